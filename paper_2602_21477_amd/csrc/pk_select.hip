// Top-k selection for gfx950: best `nprobe` centroids per query (Section 2.2, coarse
// search) and best `k` vectors per query
// over the scored candidates of all probed lists, i.e. the merge of the per-list partial
// results (Section 4.4: partial results are merged into the final result).
//
// A candidate is one 64-bit key: the value mapped to an unsigned integer whose ascending
// order is best-first (high word) and the candidate's position inside the query's
// candidate range (low word).  Keys are unique, so "smaller key" is a strict total order
// and the selection is deterministic.  A workgroup streams candidates, keeps those that
// beat the current K-th key in an LDS buffer, and re-sorts the buffer (bitonic network)
// only when it runs full, so almost all candidates cost one compare.
#include <algorithm>
#include <type_traits>

#include "pk_internal.h"
PK_DEV_MARKS(sel)
#define PK_WL_MARK(i) PK_MARK(sel, i)
#include "pk_worklist_dev.h"
#include "pk_select_dev.h"

namespace pk {

typedef unsigned long long u64;
typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t next_pow2(uint32_t n)
{
    uint32_t p = 2;
    while (p < n) p <<= 1;
    return p;
}

// ascending bitonic sort of keys[0, np2), np2 a power of two; all threads of the block call it
__device__ void bitonic_sort(u64 *keys, uint32_t np2)
{
    for (uint32_t size = 2; size <= np2; size <<= 1) {
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
            for (uint32_t i = threadIdx.x; i < (np2 >> 1); i += blockDim.x) {
                const uint32_t lo = 2 * i - (i & (stride - 1));
                const uint32_t hi = lo + stride;
                const bool up = (lo & size) == 0;
                const u64 x = keys[lo], y = keys[hi];
                if ((x > y) == up) {
                    keys[lo] = y;
                    keys[hi] = x;
                }
            }
            __syncthreads();
        }
    }
}

// Streaming selector state.  keys: LDS [cap]; cnt: LDS counter.
struct Selector {
    u64 *keys;
    uint32_t *cnt;
    int K;
    uint32_t cap; // entries of keys (a power of two >= 512)
    u64 thr;

    __device__ __forceinline__ void init(u64 *k, uint32_t *c, int kk, uint32_t capacity = (uint32_t)kSelCap)
    {
        keys = k;
        cnt = c;
        K = kk;
        cap = capacity;
        thr = kMaxKey;
        if (threadIdx.x == 0) *cnt = 0;
        __syncthreads();
    }
    // sort what is buffered, keep the best K, tighten the threshold (block-wide)
    __device__ __forceinline__ void flush()
    {
        __syncthreads();
        const uint32_t n = *cnt;
        const uint32_t np2 = next_pow2(n);
        for (uint32_t i = n + threadIdx.x; i < np2; i += blockDim.x) keys[i] = kMaxKey;
        __syncthreads();
        bitonic_sort(keys, np2);
        const uint32_t kept = n < (uint32_t)K ? n : (uint32_t)K;
        thr = kept == (uint32_t)K ? keys[K - 1] : kMaxKey;
        __syncthreads();
        if (threadIdx.x == 0) *cnt = kept;
        __syncthreads();
    }
    // make room for one round of at most `room` pushes (block-wide)
    __device__ __forceinline__ void reserve(uint32_t room)
    {
        __syncthreads();
        const uint32_t n = *cnt; // read by everyone before anyone pushes again
        __syncthreads();
        // flush threshold: the smallest power of two that holds the kept keys plus one round
        // (small rounds and small K sort small buffers)
        uint32_t limit = next_pow2((uint32_t)K + room);
        limit = limit < 512u ? 512u : (limit > cap ? cap : limit);
        if (n + room > limit) flush();
    }
    __device__ __forceinline__ void push(u64 key)
    {
        if (key < thr) keys[atomicAdd(cnt, 1u)] = key;
    }
};

__global__ __launch_bounds__(kSelThreads) void select_partial_kernel(SelectArgs a)
{
    __shared__ u64 keys[kSelCap];
    __shared__ uint32_t s_cnt;
    const uint32_t q = blockIdx.y, c = blockIdx.x;
    const uint32_t base = a.qoff[q];
    const uint32_t total = a.qcnt[q];
    const uint32_t beg = c * (uint32_t)a.chunk;
    const uint32_t end = min(beg + (uint32_t)a.chunk, total);
    // nothing in this chunk; and a query whose emitted keys fit one chunk is merged directly
    // by the final kernel
    if (beg >= total || (!a.vals && total <= (uint32_t)a.chunk)) return;
    u64 *out = a.partial + ((size_t)q * a.nchunks + c) * a.K;

    Selector sel;
    sel.init(keys, &s_cnt, a.K);
    constexpr uint32_t kRound = kSelThreads * kSelVec;
    if (a.vals) {
        const float *v = a.vals + base;
        for (uint32_t r = beg; r < end; r += kRound) {
            sel.reserve(kRound);
            const uint32_t p = r + threadIdx.x * kSelVec;
            if (p < end) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(v + p);
#pragma unroll
                for (int j = 0; j < kSelVec; ++j)
                    if (p + j < end) sel.push(((u64)order_bits(x[j], a.metric) << 32) | (p + j));
            }
        }
    } else {
        // keys were emitted under a threshold that tightened over time, so the latest are
        // the best: reading the range backwards sets a tight selection threshold at once
        const u64 *v = a.keys + base;
        for (uint32_t r = end; r > beg;) {
            const uint32_t lo = r - beg > kRound ? r - kRound : beg;
            sel.reserve(kRound);
            const uint32_t p = lo + threadIdx.x * kSelVec;
#pragma unroll
            for (int j = 0; j < kSelVec; ++j)
                if (p + j < r) sel.push(v[p + j]);
            r = lo;
        }
    }
    sel.flush();
    const uint32_t n = s_cnt;
    for (uint32_t i = threadIdx.x; i < (uint32_t)a.K; i += blockDim.x) out[i] = i < n ? keys[i] : kMaxKey;
}

// merge `nchunks` sorted partial lists of one query; leaves the best K sorted in keys[], returns count
__device__ uint32_t merge_partials(Selector &sel, const u64 *part, int nchunks, int K)
{
    const uint32_t total = (uint32_t)nchunks * (uint32_t)K;
    for (uint32_t r = 0; r < total; r += kSelThreads) {
        sel.reserve(kSelThreads);
        const uint32_t p = r + threadIdx.x;
        if (p < total) {
            const u64 key = part[p];
            if (key != kMaxKey) sel.push(key);
        }
    }
    sel.flush();
    return *sel.cnt;
}

__global__ __launch_bounds__(kSelThreads) void select_probes_kernel(const u64 *partial, int nchunks, int K, int nprobe,
                                                                    int32_t *probes)
{
    __shared__ u64 keys[kSelCap];
    __shared__ uint32_t s_cnt;
    const uint32_t q = blockIdx.x;
    Selector sel;
    sel.init(keys, &s_cnt, K);
    merge_partials(sel, partial + (size_t)q * nchunks * K, nchunks, K);
    for (int r = threadIdx.x; r < nprobe; r += blockDim.x) probes[(size_t)q * nprobe + r] = (int32_t)(uint32_t)keys[r];
}


// ---------------------------------------------------------------- dense rows (coarse search)

// Best K of a row of n <= 256 * VPT scores (Section 2.2: the top-nprobe clusters), for the
// coarse step and for the top-1 assignment of inserts and the build.  Every thread keeps
// VPT keys in registers; the exact K-th smallest key is found digit by digit (four 8-bit
// radix passes over a 256-bin LDS histogram), then the keys below it and as many of the keys
// equal to it as are needed, lowest positions first, are collected and sorted.  Positions
// are list numbers, so ties go to the lower list number.
// GO_ON: the workgroup goes on to do its query's share of the work-list construction (kCount: pairs per list,
// candidate layout, sample tiles; kLay, kLayCut: all of it), which saves the launch that would otherwise follow the selection.
enum GoOn { kStop, kCount, kLay, kLayCut };
// keys that the selection of K probes holds in LDS: 256 within a bound, or K and what rounds them up to a power of two; two of padding
__device__ __host__ __forceinline__ uint32_t dense_keys(uint32_t K) { return (K <= 256u ? 256u : K <= 512u ? 512u : 1024u) + 2u; }
static size_t dense_lds(uint32_t K, GoOn go_on)
{
    const size_t wl = go_on == kCount ? WlCountLds::bytes(K) : go_on == kLay || go_on == kLayCut ? WlLayLds::bytes(K) : 0;
    return 4096 + dense_keys(K) * sizeof(u64) + K * sizeof(int32_t) + wl;
}
template <int VPT, GoOn GO_ON>
__global__ __launch_bounds__(256) void select_dense_kernel(const float *vals, const uint32_t *qoff, const uint32_t *qcnt,
                                                           const float *add, int metric, int K, int32_t *probes, WorklistArgs wa,
                                                           SampleArgs sm, MultiArgs ma)
{
    __shared__ uint32_t s_w[4];
    __shared__ uint32_t s_n;
    extern __shared__ __align__(16) unsigned char s_dyn[]; // (see dense_lds)
    uint32_t(*hist)[256] = reinterpret_cast<uint32_t(*)[256]>(s_dyn); // [4][256] one histogram per radix pass: zeroed once
    u64 *const sel = reinterpret_cast<u64 *>(s_dyn + 4096);            // [dense_keys(K)]
    constexpr bool COUNT = GO_ON != kStop;
    int32_t *const s_probe = reinterpret_cast<int32_t *>(sel + dense_keys((uint32_t)K)); // [K]
    [[maybe_unused]] std::conditional_t<GO_ON == kCount, WlCountLds, std::conditional_t<GO_ON == kLay || GO_ON == kLayCut, WlLayLds, uint32_t>> s_wl;
    if constexpr (COUNT) s_wl.carve(reinterpret_cast<uint32_t *>(s_probe + K), (uint32_t)K);
    PK_MARK(sel, 0);
    const uint32_t q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t n = qcnt[q];
    const float *v = vals + qoff[q];
    const float own = add ? add[q] : 0.f;
    WlIndexView view{};
    if constexpr (COUNT) view = wl_index_view(wa, ma, q); // these loads are over by the time the count needs them
    uint32_t key[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const uint32_t p = tid + 256u * j;
        float x = v[p < n ? p : 0u];
        if (add) x = fmaxf(x + own, 0.f);
        key[j] = p < n ? order_bits(x, metric) : 0xffffffffu;
    }
    if (tid == 0) s_n = 0;
    bool live[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) live[j] = tid + 256u * j < n;
    PK_MARK(sel, 1);
    // few probes of many lists: the scores within a bound on the K-th best, put in order by counting
    bool done = false;
    if (K <= (int)kMostParts) {
        uint32_t bound = 0xffffffffu;
        if (n > 256u) {
            uint32_t least = key[0];
#pragma unroll
            for (int j = 1; j < VPT; ++j) least = min(least, key[j]);
            bound = bound_of_parts(least, (uint32_t)K, hist[0]);
        } else {
            __syncthreads(); // (s_n)
        }
#pragma unroll
        for (int j = 0; j < VPT; ++j)
            if (live[j] && key[j] <= bound) {
                const uint32_t at = atomicAdd(&s_n, 1u);
                if (at < 256u) sel[at] = ((u64)key[j] << 32) | (tid + 256u * j);
            }
        __syncthreads();
        const uint32_t within = s_n;
        if (within <= 256u) { // (the same for the whole workgroup)
            if (tid < 2) sel[within + tid] = kMaxKey; // padding: the keys are read in pairs
            __syncthreads();
            if (tid < within) {
                const u64 mine = sel[tid];
                const uint32_t rank = rank_among(sel, within, mine);
                if (rank < (uint32_t)K) {
                    if constexpr (COUNT) s_probe[rank] = (int32_t)(uint32_t)mine; // the count stores the list, after its loads
                    else probes[(size_t)q * K + rank] = (int32_t)(uint32_t)mine;
                }
            }
            done = true;
        } else { // equal scores are the rule
            __syncthreads();
            if (tid == 0) s_n = 0;
        }
    }
    if (!done) {
    uint32_t krem, ties;
    const uint32_t prefix = radix_kth<VPT>(key, live, (uint32_t)K, hist, krem, ties);
    PK_MARK(sel, 2);
    // prefix is the K-th smallest key; krem of the `ties` keys equal to it are needed
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const uint32_t p = tid + 256u * j;
        if (p < n && (key[j] < prefix || (key[j] == prefix && ties == krem)))
            sel[atomicAdd(&s_n, 1u)] = ((u64)key[j] << 32) | p;
    }
    if (ties != krem) { // more equal keys than needed: take them in position order
        uint32_t taken = 0;
        for (int j = 0; j < VPT && taken < krem; ++j) { // position = tid + 256 j: ascending in j, then tid
            const uint32_t p = tid + 256u * j;
            const bool tie = p < n && key[j] == prefix;
            const unsigned long long m = __ballot(tie);
            if (lane == 0) s_w[wave] = (uint32_t)__popcll(m);
            __syncthreads();
            uint32_t rank = taken + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            for (uint32_t w = 0; w < wave; ++w) rank += s_w[w];
            const uint32_t total = s_w[0] + s_w[1] + s_w[2] + s_w[3];
            if (tie && rank < krem) sel[atomicAdd(&s_n, 1u)] = ((u64)prefix << 32) | p;
            taken += total;
            __syncthreads();
        }
    }
    if (tid < 2) sel[K + tid] = kMaxKey; // padding: the rank count reads pairs
    __syncthreads();
    PK_MARK(sel, 3);
    if (K <= 256) {
        // rank of each selected key among the K of them (keys are unique): its place in the probe list
        if (tid < (uint32_t)K) {
            const u64 mine = sel[tid];
            const uint32_t rank = rank_among(sel, (uint32_t)K, mine);
            if constexpr (COUNT) s_probe[rank] = (int32_t)(uint32_t)mine; // the count stores the list, after its loads
            else probes[(size_t)q * K + rank] = (int32_t)(uint32_t)mine;
        }
    } else {
        const uint32_t np2 = next_pow2((uint32_t)K);
        for (uint32_t i = (uint32_t)K + tid; i < np2; i += 256) sel[i] = kMaxKey;
        __syncthreads();
        bitonic_sort(sel, np2);
        for (uint32_t r = tid; r < (uint32_t)K; r += 256) {
            if constexpr (COUNT) s_probe[r] = (int32_t)(uint32_t)sel[r];
            else probes[(size_t)q * K + r] = (int32_t)(uint32_t)sel[r];
        }
    }
    } // !done
    PK_MARK(sel, 4);
    if constexpr (COUNT) {
        __syncthreads(); // the probe list is in s_probe
        if constexpr (GO_ON == kCount) wl_count_query(wa, sm, ma, q, s_wl, s_probe, probes + (size_t)q * K, view);
        if constexpr (GO_ON == kLay) wl_lay_query<false>(wa, ma, q, s_wl, s_probe, probes + (size_t)q * K, view);
        if constexpr (GO_ON == kLayCut) wl_lay_query<true>(wa, ma, q, s_wl, s_probe, probes + (size_t)q * K, view);
        PK_MARK(sel, 7);
    }
}

hipError_t launch_select_dense(const float *vals, const uint32_t *qoff, const uint32_t *qcnt, uint32_t max_cnt, int metric,
                               int K, int64_t nq, int32_t *probes, hipStream_t s, const WorklistArgs *wa, const SampleArgs *sm,
                               const MultiArgs *ma, const float *add)
{
    if (nq <= 0) return hipSuccess;
    if (max_cnt > (uint32_t)kDenseSelectMax || K > PK_MAX_NPROBE) return hipErrorInvalidValue;
    const dim3 g((uint32_t)nq), b(256);
    if (wa && (!sm || !ma || wa->nprobe != K)) return hipErrorInvalidValue;
    WorklistArgs w0{};
    SampleArgs s0{};
    MultiArgs m0;
    m0.n = 0;
    auto go = [&](auto vpt) {
        constexpr int VPT = decltype(vpt)::value;
        auto run = [&](auto kernel, GoOn go_on) {
            hipLaunchKernelGGL(kernel, g, b, dense_lds((uint32_t)K, go_on), s, vals, qoff, qcnt, add, metric, K, probes, wa ? *wa : w0, wa ? *sm : s0, wa ? *ma : m0);
        };
        if (!wa) run(select_dense_kernel<VPT, kStop>, kStop);
        else if (wa->width == 0) run(select_dense_kernel<VPT, kCount>, kCount);
        else if (wa->tile_rows == 0) run(select_dense_kernel<VPT, kLay>, kLay);
        else run(select_dense_kernel<VPT, kLayCut>, kLayCut);
    };
    if (max_cnt <= 1024) go(std::integral_constant<int, 4>{});
    else if (max_cnt <= 4096) go(std::integral_constant<int, 16>{});
    else go(std::integral_constant<int, 32>{});
    return hipGetLastError();
}

// position inside the query's candidate range -> id stored in the list page
__device__ __forceinline__ int64_t resolve_id(const FinalArgs &a, const MultiArgs &h, uint32_t q, uint32_t pos)
{
    const uint32_t *po = a.pair_off + (size_t)q * (a.nprobe + 1);
    int lo = 0, hi = a.nprobe - 1;
    while (lo < hi) { // largest r with po[r] <= pos
        const int mid = (lo + hi + 1) >> 1;
        if (po[mid] <= pos) lo = mid;
        else hi = mid - 1;
    }
    const uint32_t row = pos - po[lo];
    const uint32_t list = (uint32_t)a.probes[(size_t)q * a.nprobe + lo];
    const DevIndex &ix = *h.ix[a.qagent[q]];
    const uint32_t lp = row / (uint32_t)ix.P;
    const uint32_t pg = phys_page(ix, list, lp);
    const Arena &ar = arena_of(ix, pg);
    return ar.ids[(size_t)(pg - ar.first_page) * ix.P + (row - lp * ix.P)];
}


// the same with the query's rows of pair_off and probes in LDS, and the build-time extents of the probed lists
__device__ __forceinline__ int64_t resolve_id_lds(int nprobe, const DevIndex &ix, uint32_t pos, const uint32_t *po, const uint32_t *pr,
                                  const uint32_t *mp, const uint32_t *mb)
{
    int lo = 0, hi = nprobe - 1;
    while (lo < hi) { // largest r with po[r] <= pos
        const int mid = (lo + hi + 1) >> 1;
        if (po[mid] <= pos) lo = mid;
        else hi = mid - 1;
    }
    const uint32_t row = pos - po[lo];
    const uint32_t lp = row / (uint32_t)ix.P;
    const uint32_t pg = lp < mp[lo] ? mb[lo] + lp : ix.dtab[(size_t)pr[lo] * ix.max_dp + (lp - mp[lo])];
    const Arena &ar = arena_of(ix, pg);
    return ar.ids[(size_t)(pg - ar.first_page) * ix.P + (row - lp * ix.P)];
}

// buffer of the final selection: K kept keys plus the largest round pushed at once, as a power of two
static uint32_t final_cap(int K)
{
    uint32_t c = 512;
    while (c < (uint32_t)K + (uint32_t)(kSelThreads * kSelVec) && c < (uint32_t)kSelCap) c <<= 1;
    return c;
}

// One query (LDS: the row, then a row of zeros; qbase = the lane's part) against 32 rows of a page, 16 columns in
// each accumulator: the MFMA sequence of the scan kernels (the query in MFMA row 0, zeros in the other rows), so the
// values are bit-identical to the scan's.  Element 0 of lanes 0..15 holds the dot products.
template <int STORAGE>
__device__ __forceinline__ void score_32_rows(f32x4 &acc0, f32x4 &acc1, const char *qbase, gbytes p0, int row_bytes)
{
    const int nit = row_bytes / kIterBytes;
    const gbytes p1 = p0 + (size_t)16 * row_bytes;
    acc0 = f32x4{0.f, 0.f, 0.f, 0.f};
    acc1 = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < nit; ++it) {
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            const u32x4 qa = *reinterpret_cast<const u32x4 *>(qbase + (size_t)it * kIterBytes + s4 * 64);
            const u32x4 x0 = *reinterpret_cast<gvec4>(p0 + (size_t)it * kIterBytes + s4 * 64);
            const u32x4 x1 = *reinterpret_cast<gvec4>(p1 + (size_t)it * kIterBytes + s4 * 64);
            mfma_step<STORAGE>(acc0, qa, x0);
            mfma_step<STORAGE>(acc1, qa, x1);
        }
    }
}

// Exact pass over every row the query probes, for a query whose emission region overflowed
// (more candidates passed the gate than the region holds: no usable threshold, or a tie group
// larger than the region) and that launch_rescue did not select from (no region, or one that
// overflowed as well).  One workgroup walks the probed lists page by page; each wave scores 32 rows.
//   by_id false: every value goes to the selector as (value key, position)  -> best K
//   by_id true:  the ids of the rows whose value key equals `tau` go to the selector
//                (lowest ids of a tie group; several rows may carry one id)
// s_q: LDS, the query row then a row of zeros, qstride bytes apart.
template <int STORAGE>
__device__ void rescore_query(const FinalArgs &a, const MultiArgs &h, uint32_t q, const char *s_q, int qstride,
                              Selector &sel, bool by_id, uint32_t tau)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ln = lane & 15, lg = lane >> 4;
    const DevIndex &ix = *h.ix[a.qagent[q]];
    const int row_bytes = a.row_bytes;
    const uint32_t P = (uint32_t)ix.P;
    const float qn = a.qnorm[q];
    const uint32_t *po = a.pair_off + (size_t)q * (a.nprobe + 1);
    const char *qbase = s_q + (size_t)(ln == 0 ? 0 : 1) * qstride + lg * 16;
    for (int r = 0; r < a.nprobe; ++r) {
        const uint32_t l = (uint32_t)a.probes[(size_t)q * a.nprobe + r];
        if (l >= (uint32_t)ix.nlist) continue;
        const uint32_t len = ix.list_len[l];
        for (uint32_t lp = 0; lp * P < len; ++lp) {
            const uint32_t pg = phys_page(ix, l, lp);
            const Arena &ar = arena_of(ix, pg);
            const size_t local = (size_t)(pg - ar.first_page) * P;
            const gbytes px = in_global(ar.vec + local * (size_t)row_bytes);
            const uint32_t nrows = len - lp * P < P ? len - lp * P : P;
            for (uint32_t rb0 = 0; rb0 < nrows; rb0 += 4 * kRowBlock) {
                sel.reserve(4 * kRowBlock);
                const uint32_t rb = rb0 + (uint32_t)wave * kRowBlock;
                if (rb >= nrows) continue; // the next reserve() is a barrier every wave reaches
                // rows rb .. rb + 31 lie inside the page (its size is a multiple of 32); those past
                // nrows hold stale bytes and their values are not used
                f32x4 acc0, acc1;
                score_32_rows<STORAGE>(acc0, acc1, qbase, px + (size_t)(rb + ln) * row_bytes + lg * 16, row_bytes);
                if (lg == 0) { // accumulator element 0 of lanes 0..15: MFMA row 0 (the query) x column ln (the row)
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt) {
                        const uint32_t row = rb + (uint32_t)nt * 16u + (uint32_t)ln;
                        if (row >= nrows) continue;
                        float v = nt == 0 ? acc0[0] : acc1[0];
                        if (a.metric == PK_METRIC_L2) v = l2_from_dot(ar.norm[local + row], v, qn);
                        const uint32_t bits = order_bits(v, a.metric);
                        if (!by_id) {
                            sel.push(((u64)bits << 32) | (po[r] + lp * P + row));
                        } else if (bits == tau) {
                            sel.push((u64)ar.ids[local + row] ^ 0x8000000000000000ull); // order of signed ids
                        }
                    }
                }
            }
        }
    }
}

// Queries whose emission region overflowed, scored again by the whole chip.  The keys that a region did keep are
// candidates of the query, so the k-th best of any k of them bounds the k-th best of all; and where the scan counted
// what it emitted per bucket, stored or not, the first bucket at which the count reaches k bounds it too (a region
// that filled up with the rows of far lists before the near ones were scanned has a loose k-th best).  With both as
// the threshold every probed row is scored once more, and the few hundred that pass go to a region of their own.
// Workgroup b serves overflowed query b % n (n of them, counted by every workgroup for itself) and takes every
// n-th-workgroup's share of its pages.  Bound by latency: a query of 148 000 rows of 1536 bytes (228 MB) takes its
// 1170 pages to 512 workgroups, where select_final's one workgroup (rescore_query) needed 15.4 ms for it: a batch of
// 1024 over 10 M x 768 fp16 rows with one such query went from 18.1 to 2.96 ms, as long as one with none.
template <int STORAGE>
__global__ __launch_bounds__(kSelThreads) void rescue_kernel(FinalArgs a, MultiArgs h, uint32_t nq)
{
    extern __shared__ __align__(16) unsigned char s_dyn[];
    __shared__ __align__(16) uint32_t hist[4][256];
    __shared__ uint32_t s_wave[17];
    __shared__ uint32_t s_over[kRescueRegions]; // the overflowed queries, ascending
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // (usually there is none: one round of loads and one barrier say so)
    bool any = false;
    for (uint32_t q = (uint32_t)tid; q < nq; q += kSelThreads) any = any || a.qcnt[q] > a.ecap;
    if (!__syncthreads_or(any)) return;
    // the overflowed queries, in query order
    uint32_t n = 0;
    for (uint32_t q0 = 0; q0 < nq && n < a.rregions; q0 += kSelThreads) {
        const uint32_t q = q0 + (uint32_t)tid;
        const bool over = q < nq && a.qcnt[q] > a.ecap;
        const unsigned long long m = __ballot(over);
        __syncthreads(); // s_wave of the round before is no longer read
        if (lane == 0) s_wave[wave] = (uint32_t)__popcll(m);
        __syncthreads();
        uint32_t at = n + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        for (int w = 0; w < 4; ++w) {
            if (w < wave) at += s_wave[w];
            n += s_wave[w];
        }
        if (over && at < a.rregions) s_over[at] = q;
    }
    n = n < a.rregions ? n : a.rregions;
    if (n == 0) return;
    __syncthreads();
    const uint32_t region = blockIdx.x % n, part = blockIdx.x / n, parts = (gridDim.x - region + n - 1) / n;
    const uint32_t q = s_over[region];
    const DevIndex &ix = *h.ix[a.qagent[q]];
    const uint32_t P = (uint32_t)ix.P, nprobe = (uint32_t)a.nprobe;
    const int row_bytes = a.row_bytes, qstride = row_bytes + kQPadBytes;
    char *s_q = reinterpret_cast<char *>(s_dyn);                          // the query row, then a row of zeros
    uint32_t *s_len = reinterpret_cast<uint32_t *>(s_q + 2 * qstride);    // [nprobe] rows of each probed list
    uint32_t *s_list = s_len + nprobe, *s_page0 = s_list + nprobe;        // [nprobe] the list; [nprobe] pages before it
    for (int i = tid; i < 2 * qstride / 16; i += kSelThreads) {
        u32x4 w = {0u, 0u, 0u, 0u};
        if (i < row_bytes / 16) w = *reinterpret_cast<const u32x4 *>(a.qs + (size_t)q * row_bytes + (size_t)i * 16);
        *reinterpret_cast<u32x4 *>(s_q + (size_t)i * 16) = w;
    }
    for (uint32_t r = (uint32_t)tid; r < nprobe; r += kSelThreads) {
        const uint32_t l = (uint32_t)a.probes[(size_t)q * nprobe + r];
        const uint32_t len = l < (uint32_t)ix.nlist ? ix.list_len[l] : 0u;
        s_list[r] = l;
        s_len[r] = len;
        s_page0[r] = (len + P - 1) / P;
    }
    // threshold: the k-th best of the keys stored last (the gate tightened over time, so those are the best)
    constexpr int VPT = (int)kRescueCap / kSelThreads;
    const uint32_t used = a.ecap < kRescueCap ? a.ecap : kRescueCap; // >= k: a region holds at least k + 1 keys
    const u64 *stored = a.keys + (size_t)q * a.ecap + (a.ecap - used);
    uint32_t key[VPT];
    bool live[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const uint32_t p = (uint32_t)tid + (uint32_t)kSelThreads * j;
        live[j] = p < used;
        key[j] = live[j] ? (uint32_t)(stored[p] >> 32) : 0xffffffffu;
    }
    uint32_t left, ties;
    const uint32_t tau = radix_kth<VPT>(key, live, (uint32_t)a.k, hist, left, ties); // its barriers publish the LDS arrays
    const uint32_t pages = block_exscan(s_page0, s_page0, nprobe, s_wave);
    uint32_t bmax = (uint32_t)kHistBins - 1u; // buckets beyond this are cut (every wave works it out for itself)
    float lo_value = 0.f, inv = 0.f;
    if (a.hist) {
        static_assert(kHistBins == 64, "a lane per bucket");
        uint32_t x = a.hist[(size_t)q * kHistBins + lane];
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off);
            if (lane >= off) x += y;
        }
        const unsigned long long m = __ballot(x >= (uint32_t)a.k);
        if (m) bmax = (uint32_t)__ffsll(m) - 1u;
        lo_value = a.tlo[q];
        inv = a.tinv[q];
    }

    const int ln = lane & 15, lg = lane >> 4;
    const float qn = a.qnorm[q];
    const char *qbase = s_q + (size_t)(ln == 0 ? 0 : 1) * qstride + lg * 16;
    u64 *out = a.rkeys + (size_t)region * a.rcap;
    for (uint32_t u = part; u < pages; u += parts) {
        uint32_t lo = 0, hi = nprobe - 1; // the last list whose pages start at or before u (empty lists share a start: the last has them)
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (s_page0[mid] <= u) lo = mid;
            else hi = mid - 1;
        }
        const uint32_t lp = u - s_page0[lo], len = s_len[lo];
        const uint32_t pg = phys_page(ix, s_list[lo], lp);
        const Arena &ar = arena_of(ix, pg);
        const size_t local = (size_t)(pg - ar.first_page) * P;
        const gbytes px = in_global(ar.vec + local * (size_t)row_bytes);
        const uint32_t nrows = len - lp * P < P ? len - lp * P : P;
        const uint32_t first = a.pair_off[(size_t)q * (nprobe + 1) + lo] + lp * P; // position of the page's first row
        // rows rb .. rb + 31 lie inside the page (its size is a multiple of 32); those past nrows hold stale bytes
        // and their values are not used
        for (uint32_t rb = (uint32_t)wave * kRowBlock; rb < nrows; rb += 4 * kRowBlock) {
            f32x4 acc0, acc1;
            score_32_rows<STORAGE>(acc0, acc1, qbase, px + (size_t)(rb + ln) * row_bytes + lg * 16, row_bytes);
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const uint32_t row = rb + (uint32_t)nt * 16u + (uint32_t)ln;
                const bool mine = lg == 0 && row < nrows;
                float v = nt == 0 ? acc0[0] : acc1[0];
                if (a.metric == PK_METRIC_L2) v = l2_from_dot(mine ? ar.norm[local + row] : 0.f, v, qn);
                const uint32_t bits = order_bits(v, a.metric);
                const bool pass = mine && bits <= tau && (!a.hist || bucket_of(v, lo_value, inv, a.metric) <= bmax);
                const uint32_t m = (uint32_t)__ballot(pass); // lanes 0..15
                if (m == 0u) continue;
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(&a.rcnt[q], (uint32_t)__popc(m));
                base = __shfl(base, 0);
                const uint32_t at = base + (uint32_t)__popc(m & ((1u << ln) - 1u));
                if (pass && at < a.rcap) out[at] = ((u64)bits << 32) | (first + row);
            }
        }
    }
}

// Best K of cnt_q <= 256 * VPT keys, held in registers: the K-th smallest value by
// radix selection; among the keys with that value, if not all of them are needed, the lowest positions by a
// second selection over the low words.  The kept keys end up sorted in keys[0, min(K, cnt_q)); *s_cnt is
// their number.  get(j, p): key number p, the thread's j-th.  hist: LDS [4][256].
template <int VPT, typename G>
__device__ __forceinline__ void final_by_radix(G get, uint32_t cnt_q, uint32_t K, uint32_t (*hist)[256], u64 *keys, uint32_t *s_cnt)
{
    const uint32_t tid = threadIdx.x;
    u64 k64[VPT];
    uint32_t hi[VPT];
    bool live[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const uint32_t p = tid + (uint32_t)kSelThreads * j;
        live[j] = p < cnt_q;
        k64[j] = live[j] ? get(j, p) : kMaxKey;
        hi[j] = (uint32_t)(k64[j] >> 32);
    }
    if (tid == 0) *s_cnt = 0;
    uint32_t prefix = 0xffffffffu, lo_max = 0xffffffffu; // everything is kept
    if (cnt_q > K) {
        uint32_t left, ties;
        prefix = radix_kth<VPT>(hi, live, K, hist, left, ties);
        if (ties != left) { // block-uniform: only the `left` lowest positions of the boundary value are kept
            uint32_t lo[VPT];
            bool tl[VPT];
#pragma unroll
            for (int j = 0; j < VPT; ++j) {
                lo[j] = (uint32_t)k64[j];
                tl[j] = live[j] && hi[j] == prefix;
            }
            __syncthreads(); // the histograms are read no more
            uint32_t l2, t2;
            lo_max = radix_kth<VPT>(lo, tl, left, hist, l2, t2);
        }
    } else {
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < VPT; ++j)
        if (live[j] && (hi[j] < prefix || (hi[j] == prefix && (uint32_t)k64[j] <= lo_max))) keys[atomicAdd(s_cnt, 1u)] = k64[j];
    __syncthreads();
    const uint32_t n = *s_cnt;
    if (n <= (uint32_t)kSelThreads) {
        // order by counting: the rank of a key is the number of smaller ones (keys are unique)
        if (tid < 2) keys[n + tid] = kMaxKey; // padding: the keys are read in pairs
        __syncthreads();
        const u64 mine = tid < n ? keys[tid] : kMaxKey;
        const uint32_t rank = tid < n ? rank_among(keys, n, mine) : 0u;
        __syncthreads();
        if (tid < n) keys[rank] = mine;
        __syncthreads();
    } else {
        const uint32_t np2 = next_pow2(n);
        for (uint32_t i = n + tid; i < np2; i += blockDim.x) keys[i] = kMaxKey;
        __syncthreads();
        bitonic_sort(keys, np2);
    }
}

// A bound on the K-th smallest (K up to 256) of what the workgroup's threads met: mn[]: each thread's smallest keys of four
// parts of it, all ones for a part with none; `all`: every thread has met something.  FAR: neighbouring threads met neighbours.
template <bool FAR>
__device__ __forceinline__ uint32_t bound_on_kth(u32x4 mn, bool all, uint32_t K, uint32_t (*hist)[256])
{
    if (FAR && K <= kFewParts) return bound_of_far_parts(min(min(mn[0], mn[1]), min(mn[2], mn[3])), K, hist[0]);
    if (K <= kMostParts) return bound_of_parts(min(min(mn[0], mn[1]), min(mn[2], mn[3])), K, hist[0]);
    if (!all) return 0xffffffffu;
    const uint32_t key[4] = {mn[0], mn[1], mn[2], mn[3]};
    const bool live[4] = {key[0] != 0xffffffffu, key[1] != 0xffffffffu, key[2] != 0xffffffffu, key[3] != 0xffffffffu};
    uint32_t left, ties;
    return radix_kth<4>(key, live, K, hist, left, ties);
}

// The same of all cnt_q values of a query's range (DENSE calls): a bound on the K-th best by parts, and the few values within
// it, collected in surv and put in order by counting.  Ranges of up to kReadOnce values are read once, into registers; of
// longer ones the best keys of every 16 values are, and then only those 16 that have one within the bound: a whole search
// of one query over 250 000 values (1 M x 64, 64 lists, 16 probes) in 64 us, 124 with the values read twice, 80 gated.
// False: more than fit are within the bound, or K is too large; nothing is selected.  n_surv: how many keys surv holds, every one that is no worse than the K-th best among them (0: none).
constexpr uint32_t kBlocks = 1024;
// Keys that surv holds.  Where the query's nearest list has less than K parts' worth of values, all of it is within the
// bound, and some from other lists: a part is 4 neighbours of ranges that are read once, 16 of others, and four times that
// (of the others, from afar) where there are 64 parts.
constexpr uint32_t kMostSurvivors = 18u * kSelThreads;
__device__ __host__ __forceinline__ uint32_t survivors(uint32_t K, uint32_t width)
{
    const uint32_t want = (width <= kReadOnce ? 4u : 16u) * (K <= kFewParts ? 4u : 1u) * K + 512u;
    return want < 1024u ? 1024u : (want < kMostSurvivors ? want : kMostSurvivors);
}
__device__ __forceinline__ bool final_of_values(const float *vals, const uint32_t *mins, uint32_t width, uint32_t cnt_q, uint32_t K, int metric,
                                                uint32_t (*hist)[256], u64 *keys, u64 *surv, uint32_t &n_surv, uint32_t *s_cnt)
{
    const uint32_t tid = threadIdx.x;
    n_surv = 0;
    if (K > (uint32_t)kSelThreads) { // (the first 1024 values alone give 256 parts)
        if (cnt_q > 16u * kSelThreads) return false;
        final_by_radix<16>([=](int, uint32_t p) { return ((u64)order_bits(vals[p], metric) << 32) | p; }, cnt_q, K, hist, keys, s_cnt);
        return true;
    }
    const uint32_t room = survivors(K, width);
    constexpr int U = 8; // loads in flight
    constexpr uint32_t kStep = 4u * kSelThreads;
    static_assert(kReadOnce == U * kStep, "a round of loads");
    u32x4 v[U];
    auto load = [&](const float *from, uint32_t p0, uint32_t n) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t p = p0 + u * kStep;
            v[u] = reinterpret_cast<const u32x4 *>(from)[(p < n ? p : 0u) >> 2];
        }
    };
    u32x4 mn = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
    if (cnt_q <= kReadOnce) {
        load(vals, 4u * tid, cnt_q); // (ranges are padded to 16 values)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[u][e] = 4u * tid + u * kStep < cnt_q ? order_bits(__uint_as_float(v[u][e]), metric) : 0xffffffffu;
                mn[u & 3] = min(mn[u & 3], min(v[u][e], 0xfffffffeu) | (4u * tid + u * kStep < cnt_q ? 0u : 1u));
            }
        PK_MARK(sel, 41);
        const uint32_t bound = cnt_q > K ? bound_on_kth<false>(mn, cnt_q >= kStep, K, hist) : 0xffffffffu;
        if (cnt_q <= K) __syncthreads();
        PK_MARK(sel, 42);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t p = 4u * tid + u * kStep + e, key = v[u][e];
                if (p < cnt_q && key <= bound && key < kWorstBits) { // (padding is no candidate)
                    const uint32_t at = atomicAdd(s_cnt, 1u);
                    if (at < room) surv[at] = ((u64)key << 32) | p;
                }
            }
    } else {
        // Neighbouring blocks go to neighbouring threads: the query's nearest list lies in one piece, and where it has
        // K blocks of values or more the bound is one of theirs; where it has fewer, all of it (16 K values) and a few more
        // are within the bound.
        const uint32_t nb = cnt_q >> 4; // (more than 512)
        constexpr uint32_t V = kReadOnce / kSelThreads;
        uint32_t w[V];
        auto load_mins = [&](uint32_t r) {
#pragma unroll
            for (uint32_t u = 0; u < V; ++u) {
                const uint32_t b = r + u * kSelThreads + tid;
                w[u] = mins[b < nb ? b : 0u];
            }
        };
        for (uint32_t r = 0; r < nb; r += kReadOnce) {
            load_mins(r);
#pragma unroll
            for (uint32_t u = 0; u < V; ++u)
                if (r + u * kSelThreads + tid < nb) mn[u & 3] = min(mn[u & 3], min(w[u], 0xfffffffeu));
        }
        PK_MARK(sel, 41);
        const uint32_t bound = bound_on_kth<true>(mn, nb >= (uint32_t)kSelThreads, K, hist);
        PK_MARK(sel, 42);
        uint32_t *const blocks = reinterpret_cast<uint32_t *>(keys); // (the kept keys come later)
        for (uint32_t r = 0; r < nb; r += kReadOnce) {
            if (nb > kReadOnce) load_mins(r);
#pragma unroll
            for (uint32_t u = 0; u < V; ++u) {
                const uint32_t b = r + u * kSelThreads + tid;
                if (b < nb && w[u] <= bound && w[u] < kWorstBits) {
                    const uint32_t at = atomicAdd(s_cnt, 1u);
                    if (at < kBlocks) blocks[at] = b;
                }
            }
        }
        __syncthreads();
        const uint32_t within = *s_cnt;
        __syncthreads();
        if (within > kBlocks) return false;
        if (tid == 0) *s_cnt = 0;
        __syncthreads();
        for (uint32_t i = tid; i < within * 16u; i += 4u * kSelThreads) { // 16 threads a block, four blocks in flight
            u32x4 p;
            f32x4 x;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = i + u * kSelThreads;
                p[u] = blocks[j < within * 16u ? j >> 4 : 0u] * 16u + (j & 15u);
                x[u] = vals[p[u]];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t key = order_bits(x[u], metric);
                if (i + u * kSelThreads < within * 16u && key <= bound && key < kWorstBits) {
                    const uint32_t at = atomicAdd(s_cnt, 1u);
                    if (at < room) surv[at] = ((u64)key << 32) | p[u];
                }
            }
        }
    }
    __syncthreads();
    const uint32_t n = *s_cnt;
    PK_MARK(sel, 43);
    if (n > room) {
        __syncthreads(); // (the caller counts in the same word)
        return false;
    }
    n_surv = n;
    if (n <= (uint32_t)kSelThreads) {
        if (tid < 2) surv[n + tid] = kMaxKey; // padding: the keys are read in pairs
        __syncthreads();
        if (tid < n) {
            const u64 mine = surv[tid];
            const uint32_t rank = rank_among(surv, n, mine);
            if (rank < K) keys[rank] = mine;
        }
        if (tid == 0) *s_cnt = n < K ? n : K;
        __syncthreads();
    } else {
        __syncthreads(); // (the selection counts in the same word)
        // A bound from parts again, now of the collected keys alone: where the nearest list was too short to fill K parts, the
        // first bound was a value of some other list.  (K = 78 of lists of 370: 2 us of 19, where radix passes took 4.5.)
        if (K <= kMostParts && n <= 16u * kSelThreads) {
            uint32_t least = 0xffffffffu;
            for (uint32_t p = tid; p < n; p += kSelThreads) least = min(least, (uint32_t)(surv[p] >> 32));
            if (tid == 0) *s_cnt = 0;
            const uint32_t bound = bound_of_parts(least, K, hist[0]);
            for (uint32_t p = tid; p < n; p += kSelThreads) {
                const u64 key = surv[p];
                if ((uint32_t)(key >> 32) > bound) continue;
                const uint32_t at = atomicAdd(s_cnt, 1u);
                if (at < (uint32_t)kSelThreads) keys[at] = key;
            }
            __syncthreads();
            const uint32_t within = *s_cnt;
            __syncthreads();
            if (within <= (uint32_t)kSelThreads) { // (the same for the whole workgroup)
                if (tid < 2) keys[within + tid] = kMaxKey; // padding: the keys are read in pairs
                __syncthreads();
                const u64 mine = tid < within ? keys[tid] : kMaxKey;
                const uint32_t rank = tid < within ? rank_among(keys, within, mine) : K;
                __syncthreads();
                if (rank < K) keys[rank] = mine;
                if (tid == 0) *s_cnt = within < K ? within : K;
                __syncthreads();
                return true;
            }
        }
        if (n <= 4u * kSelThreads) final_by_radix<4>([=](int, uint32_t p) { return surv[p]; }, n, K, hist, keys, s_cnt);
        else final_by_radix<kMostSurvivors / kSelThreads>([=](int, uint32_t p) { return surv[p]; }, n, K, hist, keys, s_cnt);
    }
    return true;
}

// All n values of a query's range (aligned, padded to 16) through a selector, for queries among whose values equal ones are the
// rule.  key(bits, p): what the value with these order bits at position p is selected by, all ones for not at all, which is what
// all values have that may(bits, threshold) refuses.  A round is 8192 values, and only those 256 of it are pushed among which
// some thread has a key below the threshold.  700 000 values of
// 50 kinds: values and the ids of a group in 0.5 ms, 1 M equal ones 4.7 (gated, whose rows are scored again, 1.4 - 10 and 76).
// s_mask: LDS, zero.
template <typename May, typename Key>
__device__ __forceinline__ void stream_values(Selector &sel, uint32_t *s_mask, const float *vals, uint32_t n, int metric, May may, Key key)
{
    constexpr uint32_t U = 8, kStep = 4u * kSelThreads;
    const uint32_t tid = threadIdx.x;
    for (uint32_t r = 0; r < n; r += U * kStep) {
        u32x4 v[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t p = r + u * kStep + 4u * tid;
            v[u] = reinterpret_cast<const u32x4 *>(vals)[(p < n ? p : 0u) >> 2];
        }
        uint32_t some = 0, pass = 0;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) {
                const uint32_t p = r + u * kStep + 4u * tid + e;
                if (p < n && may(order_bits(__uint_as_float(v[u][e]), metric), sel.thr)) some |= 1u << (u * 4u + e);
            }
        // (from here on one value at a time, read again: as 32 copies of the loops' bodies this was most of the kernel's code)
        auto at = [=](uint32_t b) { return r + (b >> 2) * kStep + 4u * tid + (b & 3u); };
        for (; some != 0u; some &= some - 1u) {
            const uint32_t b = (uint32_t)__ffs(some) - 1u;
            if (key(order_bits(vals[at(b)], metric), at(b)) < sel.thr) pass |= 1u << b;
        }
        for (int off = 32; off > 0; off >>= 1) pass |= __shfl_xor(pass, off);
        if ((tid & 63u) == 0u && pass) atomicOr(s_mask, pass);
        __syncthreads();
        pass = *s_mask; // (the same for the whole workgroup)
        __syncthreads();
        if (tid == 0) *s_mask = 0u;
        for (; pass != 0u; pass &= pass - 1u) {
            const uint32_t p = at((uint32_t)__ffs(pass) - 1u);
            sel.reserve(kSelThreads);
            if (p < n) sel.push(key(order_bits(vals[p], metric), p));
        }
        __syncthreads(); // (s_mask: written again)
    }
}

template <bool DENSE>
__global__ __launch_bounds__(kSelThreads) void select_final_kernel(FinalArgs a, MultiArgs h, uint32_t cap, uint32_t qbytes)
{
    // LDS sized by K, not by the largest K the library takes: small k leaves room for every
    // query's workgroup to be resident at once
    extern __shared__ __align__(16) unsigned char s_dyn[];
    u64 *keys = reinterpret_cast<u64 *>(s_dyn);                  // [cap]
    int64_t *s_id = reinterpret_cast<int64_t *>(keys + cap);     // [k]
    // [2][row_bytes + kQPadBytes] when rescoring; the histograms of the radix selection otherwise
    char *s_q = reinterpret_cast<char *>(s_id + ((a.k + 1) & ~1));
    [[maybe_unused]] u64 *const s_surv = reinterpret_cast<u64 *>(s_q + 4 * 256 * sizeof(uint32_t)); // DENSE: behind the histograms
    uint32_t *s_po = reinterpret_cast<uint32_t *>(s_q + qbytes); // [nprobe + 1] the query's row of pair_off
    uint32_t *s_pr = s_po + a.nprobe + 1;                        // [nprobe] its probe list,
    uint32_t *s_mp = s_pr + a.nprobe, *s_mb = s_mp + a.nprobe;   // [nprobe] pages and first page of the lists' build-time extents
    __shared__ uint32_t s_cnt;
    __shared__ long long s_red[kSelThreads / 64];
    __shared__ uint32_t s_redpos[kSelThreads / 64];
    __shared__ long long s_pick;
    __shared__ uint32_t s_pickpos;
    const uint32_t q = blockIdx.x;
    const int k = a.k;
    const int qstride = a.row_bytes + kQPadBytes;
    PK_MARK(sel, 32);
    const size_t region = DENSE ? 0 : (size_t)q * a.ecap;
    // everything the usual path reads from global memory is requested at once: the count, the thread's key
    // of a short region (the entry exists whatever the count; it is used only if it is below it), the
    // query's rows of the candidate layout, its index
    uint32_t cnt_q = DENSE ? a.pair_off[(size_t)q * (a.nprobe + 1) + a.nprobe] : a.qcnt[q];
    [[maybe_unused]] bool refused = false; // the work list had no room: no query has values (cannot happen while the host bounds hold)
    if constexpr (DENSE) refused = *a.ntiles > a.tile_cap;
    u64 early = !DENSE && threadIdx.x < a.ecap ? a.keys[region + threadIdx.x] : kMaxKey;
    const DevIndex &qix = *h.ix[a.qagent[q]];
    for (int r = threadIdx.x; r <= a.nprobe; r += blockDim.x) {
        s_po[r] = a.pair_off[(size_t)q * (a.nprobe + 1) + r];
        if (r < a.nprobe) {
            const uint32_t l = (uint32_t)a.probes[(size_t)q * a.nprobe + r];
            const bool valid = l < (uint32_t)qix.nlist;
            s_pr[r] = l;
            s_mp[r] = valid ? qix.main_pages[l] : 0u;
            s_mb[r] = valid ? qix.main_base[l] : 0u;
        }
    }
    // Running sums of the call (candidates met, candidates emitted, most emitted by one query, queries whose
    // region overflowed): workgroup 0 adds up every query's numbers, so that they cost four atomics per call
    // and not several per query on the same words.
    unsigned long long st_cand = 0, st_emit = 0;
    uint32_t st_max = 0, st_over = 0;
    if (blockIdx.x == 0) {
        for (uint32_t t = threadIdx.x; t < gridDim.x; t += blockDim.x) {
            const uint32_t all = a.pair_off[(size_t)t * (a.nprobe + 1) + a.nprobe], c = DENSE ? (refused ? 0u : all) : a.qcnt[t];
            st_cand += all;
            st_emit += c;
            st_max = c > st_max ? c : st_max;
            st_over += !DENSE && c > a.ecap ? 1u : 0u;
        }
    }
    if (DENSE && refused) cnt_q = 0u;
    Selector sel;
    sel.init(keys, &s_cnt, a.K, cap);
    bool overflow = !DENSE && cnt_q > a.ecap; // the region lost candidates: select by rescoring the query's rows
    const u64 *v = a.keys + region;           // where the query's candidates are
    if (!DENSE && overflow && a.rregions > 0) {
        // ... unless they were scored again already: the query's region is its number among the overflowed queries
        uint32_t before = 0;
        for (uint32_t t = threadIdx.x; t < q; t += blockDim.x) before += a.qcnt[t] > a.ecap ? 1u : 0u;
        for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off);
        if ((threadIdx.x & 63) == 0) s_redpos[threadIdx.x >> 6] = before;
        __syncthreads();
        before = s_redpos[0] + s_redpos[1] + s_redpos[2] + s_redpos[3];
        const uint32_t got = a.rcnt[q];
        if (before < a.rregions && got <= a.rcap) {
            overflow = false;
            v = a.rkeys + (size_t)before * a.rcap;
            cnt_q = got;
            early = threadIdx.x < got ? v[threadIdx.x] : kMaxKey;
        }
    }
    bool in_registers = cnt_q <= 16u * kSelThreads && !overflow;
    uint32_t(*hist)[256] = reinterpret_cast<uint32_t(*)[256]>(s_q);
    [[maybe_unused]] const float *const values = DENSE ? a.vals + (size_t)q * a.width : nullptr;
    [[maybe_unused]] uint32_t n_surv = 0;
    if constexpr (DENSE) in_registers = final_of_values(values, a.mins ? a.mins + (size_t)q * (a.width / 16u) : nullptr, a.width, cnt_q, (uint32_t)a.K,
                                                        a.metric, hist, keys, s_surv, n_surv, &s_cnt);
    if (DENSE && !in_registers) {
        // equal values are the rule: all of them through the streaming selector
        if (threadIdx.x == 0) s_cnt = s_pickpos = 0;
        __syncthreads();
        stream_values(sel, &s_pickpos, values, cnt_q, a.metric,
                      [](uint32_t bits, u64 thr) { return bits < kWorstBits && bits <= (uint32_t)(thr >> 32); },
                      [](uint32_t bits, uint32_t p) { return bits < kWorstBits ? ((u64)bits << 32) | p : kMaxKey; });
    } else if (DENSE) {
    } else if (in_registers) {
        auto get = [=](int j, uint32_t p) { return j == 0 ? early : v[p]; };
        if (cnt_q <= (uint32_t)kSelThreads) final_by_radix<1>(get, cnt_q, (uint32_t)a.K, hist, keys, &s_cnt);
        else if (cnt_q <= 4u * kSelThreads) final_by_radix<4>(get, cnt_q, (uint32_t)a.K, hist, keys, &s_cnt);
        else final_by_radix<16>(get, cnt_q, (uint32_t)a.K, hist, keys, &s_cnt);
    } else if (!overflow) {
        // short ranges go one key per thread and round, so the buffer that gets sorted stays small
        const uint32_t per = cnt_q <= 8192u ? 1u : (uint32_t)kSelVec;
        const uint32_t round = kSelThreads * per;
        // keys were emitted under a gate that tightened over time, so the latest are the best:
        // reading the region backwards sets a tight selection threshold at once
        for (uint32_t r = cnt_q; r > 0;) {
            const uint32_t lo = r > round ? r - round : 0u;
            sel.reserve(round);
            const uint32_t p = lo + threadIdx.x * per;
            for (uint32_t j = 0; j < per; ++j)
                if (p + j < r) sel.push(v[p + j]);
            r = lo;
        }
    } else {
        // the query row (its padding zeroed), then a row of zeros
        for (int i = threadIdx.x; i < 2 * qstride / 16; i += blockDim.x) {
            u32x4 w = {0u, 0u, 0u, 0u};
            if (i < a.row_bytes / 16) w = *reinterpret_cast<const u32x4 *>(a.qs + (size_t)q * a.row_bytes + (size_t)i * 16);
            *reinterpret_cast<u32x4 *>(s_q + (size_t)i * 16) = w;
        }
        __syncthreads();
        if (a.storage == PK_F16) rescore_query<PK_F16>(a, h, q, s_q, qstride, sel, false, 0u);
        else rescore_query<PK_F32>(a, h, q, s_q, qstride, sel, false, 0u);
    }
    PK_MARK(sel, 33);
    if (!in_registers) sel.flush();
    const uint32_t n = s_cnt;

    // entries carrying the padding value are not candidates
    const uint32_t worst = kWorstBits;
    uint32_t n_valid = 0;
    for (uint32_t i = 0; i < n; i += kSelThreads) // (sorted: they come last)
        n_valid += (uint32_t)__syncthreads_count(i + threadIdx.x < n && (uint32_t)(keys[i + threadIdx.x] >> 32) < worst);
    const uint32_t kk = n_valid < (uint32_t)k ? n_valid : (uint32_t)k;
    for (uint32_t i = threadIdx.x; i < kk; i += blockDim.x) s_id[i] = resolve_id_lds(a.nprobe, qix, (uint32_t)keys[i], s_po, s_pr, s_mp, s_mb);
    __syncthreads();
    PK_MARK(sel, 34);

    // Equal values must come in ascending id order.  If the tie group of the k-th value
    // reaches past position k, its members inside the top k are the lowest ids of the
    // whole group, which may include candidates the selection above did not keep: look again.
    if (n_valid > (uint32_t)k && (uint32_t)(keys[k - 1] >> 32) == (uint32_t)(keys[k] >> 32)) {
        const uint32_t tau = (uint32_t)(keys[k - 1] >> 32);
        uint32_t nb = 0;
        while (nb < (uint32_t)k && (uint32_t)(keys[nb] >> 32) < tau) ++nb;
        if (overflow) {
            // the kept keys better than the tie value wait in the query's (unusable) region while
            // the selector collects the lowest ids of the tie group
            u64 *spill = a.spill + region;
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < nb; i += blockDim.x) spill[i] = keys[i];
            __syncthreads();
            sel.init(keys, &s_cnt, (int)((uint32_t)k - nb), cap);
            if (a.storage == PK_F16) rescore_query<PK_F16>(a, h, q, s_q, qstride, sel, true, tau);
            else rescore_query<PK_F32>(a, h, q, s_q, qstride, sel, true, tau);
            sel.flush();
            for (uint32_t t = nb + threadIdx.x; t < (uint32_t)k; t += blockDim.x)
                s_id[t] = (int64_t)(keys[t - nb] ^ 0x8000000000000000ull);
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < (uint32_t)k; t += blockDim.x)
                keys[t] = t < nb ? spill[t] : (((u64)tau << 32) | t); // the low word is no longer used
            __syncthreads();
        } else if (DENSE && !in_registers) {
            // The lowest ids of the group by one more pass over the values (one pass for each of its members in the top k
            // would be up to k of them: 700 000 values of 50 kinds, k = 100, took 31 ms); the kept keys better than the
            // tie value wait where candidates are collected otherwise.
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < nb; i += blockDim.x) s_surv[i] = keys[i];
            __syncthreads();
            sel.init(keys, &s_cnt, (int)((uint32_t)k - nb), cap);
            const DevIndex *const ix = &qix;
            const int nprobe = a.nprobe;
            stream_values(sel, &s_pickpos, values, cnt_q, a.metric, [=](uint32_t bits, u64) { return bits == tau; },
                          [=](uint32_t bits, uint32_t p) {
                              return bits == tau ? (u64)resolve_id_lds(nprobe, *ix, p, s_po, s_pr, s_mp, s_mb) ^ 0x8000000000000000ull : kMaxKey;
                          });
            sel.flush();
            for (uint32_t t = nb + threadIdx.x; t < (uint32_t)k; t += blockDim.x) // (the largest id there is has the key of none)
                s_id[t] = t - nb < s_cnt ? (int64_t)(keys[t - nb] ^ 0x8000000000000000ull) : INT64_MAX;
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < (uint32_t)k; t += blockDim.x)
                keys[t] = t < nb ? s_surv[t] : (((u64)tau << 32) | t); // the low word is no longer used
            __syncthreads();
        } else {
        const uint32_t total = n_surv > 0 ? n_surv : cnt_q;
        const int metric = a.metric;
        auto key_at = [=](uint32_t p) { // (nothing by reference: the kernel's arguments would be copied to memory)
            if constexpr (DENSE) return n_surv > 0 ? s_surv[p] : ((u64)order_bits(values[p], metric) << 32) | p;
            else return v[p];
        };
        // Members are taken in (id, position) order: several rows may carry one id, and each
        // of them is a candidate of its own.
        long long last_id = 0;
        uint32_t last_pos = 0;
        bool have_last = false;
        for (uint32_t t = nb; t < (uint32_t)k; ++t) {
            long long best = INT64_MAX;
            uint32_t best_pos = 0xffffffffu;
            for (uint32_t p = threadIdx.x; p < total; p += blockDim.x) {
                const u64 key = key_at(p);
                if ((uint32_t)(key >> 32) == tau) {
                    const uint32_t pos = (uint32_t)key;
                    const long long id = resolve_id(a, h, q, pos);
                    const bool after = !have_last || id > last_id || (id == last_id && pos > last_pos);
                    if (after && (id < best || (id == best && pos < best_pos))) {
                        best = id;
                        best_pos = pos;
                    }
                }
            }
            for (int off = 32; off > 0; off >>= 1) {
                const long long o = __shfl_xor(best, off);
                const uint32_t op = __shfl_xor(best_pos, off);
                if (o < best || (o == best && op < best_pos)) {
                    best = o;
                    best_pos = op;
                }
            }
            if ((threadIdx.x & 63) == 0) {
                s_red[threadIdx.x >> 6] = best;
                s_redpos[threadIdx.x >> 6] = best_pos;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                long long b = s_red[0];
                uint32_t bp = s_redpos[0];
                for (int w = 1; w < kSelThreads / 64; ++w)
                    if (s_red[w] < b || (s_red[w] == b && s_redpos[w] < bp)) {
                        b = s_red[w];
                        bp = s_redpos[w];
                    }
                s_pick = b;
                s_pickpos = bp;
                s_id[t] = b;
                keys[t] = ((u64)tau << 32) | (uint32_t)t; // keeps the value; the low word is no longer used
            }
            __syncthreads();
            last_id = s_pick;
            last_pos = s_pickpos;
            have_last = true;
            __syncthreads();
        }
        }
    }

    PK_MARK(sel, 35);
    // final order: (value key, id) ascending; rows that carry the same id with the same value
    // keep their order in keys[], so ranks are unique
    for (uint32_t i = threadIdx.x; i < (uint32_t)k; i += blockDim.x) {
        if (i < kk) {
            const uint32_t ki = (uint32_t)(keys[i] >> 32);
            const int64_t idi = s_id[i];
            // keys[] is sorted by (value key, position): only neighbours of the same value can change places
            uint32_t rank = i;
            for (uint32_t j = i; j > 0 && (uint32_t)(keys[j - 1] >> 32) == ki; --j) rank -= s_id[j - 1] > idi ? 1u : 0u;
            for (uint32_t j = i + 1; j < kk && (uint32_t)(keys[j] >> 32) == ki; ++j) rank += s_id[j] < idi ? 1u : 0u;
            a.out_ids[(size_t)q * k + rank] = idi;
            a.out_dist[(size_t)q * k + rank] = value_of(ki, a.metric);
        } else {
            a.out_ids[(size_t)q * k + i] = -1;
            a.out_dist[(size_t)q * k + i] = a.metric == PK_METRIC_IP ? -INFINITY : INFINITY;
        }
    }
    if (blockIdx.x == 0) { // last: no load above queues behind these atomics
        for (int off = 32; off > 0; off >>= 1) {
            st_cand += __shfl_xor(st_cand, off);
            st_emit += __shfl_xor(st_emit, off);
            const uint32_t o = __shfl_xor(st_max, off);
            st_max = o > st_max ? o : st_max;
            st_over += __shfl_xor(st_over, off);
        }
        __syncthreads(); // keys[] is no longer read
        if ((threadIdx.x & 63) == 0) {
            u64 *w = keys + 4 * (threadIdx.x >> 6);
            w[0] = st_cand;
            w[1] = st_emit;
            w[2] = st_max;
            w[3] = st_over;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            u64 cand = 0, emit = 0, mx = 0, over = 0;
            for (int w = 0; w < kSelThreads / 64; ++w) {
                cand += keys[4 * w];
                emit += keys[4 * w + 1];
                mx = keys[4 * w + 2] > mx ? keys[4 * w + 2] : mx;
                over += keys[4 * w + 3];
            }
            unsigned long long *st = h.ix[0]->stats;
            atomicAdd(&st[1], cand);
            atomicAdd(&st[3], emit);
            if (over) atomicAdd(&st[4], over);
            atomicMax(&st[5], mx);
        }
    }
}

// k-th best of each query's sample -> threshold key; fewer than k real samples: no threshold.  For samples
// scored by a launch of their own (large batches; small ones usually take sample_tau_kernel instead).
// WL: the workgroups then lay out the second half of the work list between them (offsets, slots, tiles:
// small batches whose samples are too long for the one-launch form), so that no launch of its own is
// needed for it.
template <bool WL>
__global__ __launch_bounds__(kSelThreads) void tau_kernel(SampleArgs a, WorklistArgs wa, MultiArgs ma)
{
    __shared__ __align__(16) u64 keys[kSelCap];
    __shared__ uint32_t s_cnt;
    __shared__ uint32_t s_wave[17];
    const uint32_t q = blockIdx.x;
    PK_MARK(sel, 16);
    WlPrefetch pre;
    auto read_ahead = [&]() {
        if constexpr (WL) wl_spread_prefetch(wa, ma, q, pre); // in flight while the threshold is worked out
    };
    const float *v = a.vals + (size_t)q * a.span;
    uint32_t cnt = 0;                      // real samples (or k, if there are more)
    uint32_t first = 0, kth = 0, last = 0; // value keys: best, k-th best, worst real sample
    uint32_t(*hist)[256] = reinterpret_cast<uint32_t(*)[256]>(keys);
    if (a.span <= 4u * kSelThreads) {
        tau_by_radix<4>(a, v, hist, s_wave, cnt, first, kth, last, read_ahead);
    } else if (a.span <= 16u * kSelThreads) {
        tau_by_radix<16>(a, v, hist, s_wave, cnt, first, kth, last, read_ahead);
    } else {
        read_ahead();
        Selector sel;
        sel.init(keys, &s_cnt, a.k);
        constexpr uint32_t kRound = kSelThreads * kSelVec;
        for (uint32_t r = 0; r < a.span; r += kRound) {
            sel.reserve(kRound);
            const uint32_t p = r + threadIdx.x * kSelVec;
            if (p < a.span) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(v + p);
#pragma unroll
                for (int j = 0; j < kSelVec; ++j) {
                    const uint32_t b = order_bits(x[j], a.metric);
                    if (b < kWorstBits) sel.push(((u64)b << 32) | (p + j));
                }
            }
        }
        sel.flush();
        cnt = s_cnt; // at most k are kept
        if (cnt > 0) {
            first = (uint32_t)(keys[0] >> 32);
            last = (uint32_t)(keys[cnt - 1] >> 32);
            kth = last;
        }
    }
    PK_MARK(sel, 18);
    if constexpr (WL) {
        __syncthreads(); // the key buffer is free
        wl_spread(wa, ma, reinterpret_cast<uint32_t *>(keys), s_wave, q, pre);
        PK_MARK(sel, 24);
    }
    // the kernel's own results last: no load above queues behind these stores
    tau_publish(a, q, cnt, first, kth, last);
}

hipError_t launch_tau(const SampleArgs &a, hipStream_t s, const WorklistArgs *wa, const MultiArgs *ma)
{
    if (a.nq <= 0) return hipSuccess;
    if (a.span % 4 != 0) return hipErrorInvalidValue;
    if (wa) {
        static_assert(2 * kSelCap >= 3 * ((int)kWlSmallLists + 1), "the work-list layout borrows the key buffer");
        static_assert(kSelThreads * 8 >= (int)kWlSmallLists, "one round of the list scan covers every list");
        if (!ma || (uint64_t)wa->n_handles * (uint64_t)wa->nlist_max > kWlSmallLists) return hipErrorInvalidValue;
        hipLaunchKernelGGL(tau_kernel<true>, dim3((uint32_t)a.nq), dim3(kSelThreads), 0, s, a, *wa, *ma);
        return hipGetLastError();
    }
    MultiArgs m0;
    m0.n = 0;
    hipLaunchKernelGGL(tau_kernel<false>, dim3((uint32_t)a.nq), dim3(kSelThreads), 0, s, a, WorklistArgs{}, m0);
    return hipGetLastError();
}

hipError_t launch_select_partial(const SelectArgs &a, int64_t nq, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    hipLaunchKernelGGL(select_partial_kernel, dim3(a.nchunks, (uint32_t)nq), dim3(kSelThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_select_probes(const unsigned long long *partial, int nchunks, int K, int nprobe, int64_t nq,
                                int32_t *probes, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    hipLaunchKernelGGL(select_probes_kernel, dim3((uint32_t)nq), dim3(kSelThreads), 0, s, partial, nchunks, K, nprobe,
                       probes);
    return hipGetLastError();
}

// grid: workgroups (at least rregions)
hipError_t launch_rescue(const FinalArgs &a, const MultiArgs &m, int64_t nq, int grid, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    static_assert(kRescueCap % kSelThreads == 0, "the threshold of a rescue comes out of registers");
    if (a.row_bytes <= 0 || a.row_bytes % kIterBytes != 0 || a.ecap < (uint32_t)a.K || a.rcap != kRescueCap ||
        a.rregions < 1 || a.rregions > kRescueRegions || grid < (int)a.rregions)
        return hipErrorInvalidValue;
    const size_t lds = (size_t)2 * (a.row_bytes + kQPadBytes) + (size_t)3 * a.nprobe * sizeof(uint32_t);
    if (a.storage == PK_F16)
        hipLaunchKernelGGL(rescue_kernel<PK_F16>, dim3(grid), dim3(kSelThreads), lds, s, a, m, (uint32_t)nq);
    else
        hipLaunchKernelGGL(rescue_kernel<PK_F32>, dim3(grid), dim3(kSelThreads), lds, s, a, m, (uint32_t)nq);
    return hipGetLastError();
}

hipError_t launch_select_final(const FinalArgs &a, const MultiArgs &h, int64_t nq, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    const bool dense = a.vals != nullptr;
    if (a.row_bytes <= 0 || a.row_bytes % kIterBytes != 0 || (!dense && a.ecap < (uint32_t)a.K)) return hipErrorInvalidValue;
    if (dense && (a.width % 64 != 0 || (reinterpret_cast<uintptr_t>(a.vals) & 15) != 0 || (a.width > kReadOnce && !a.mins) ||
                  (reinterpret_cast<uintptr_t>(a.mins) & 15) != 0))
        return hipErrorInvalidValue;
    // (dense calls buffer a round of one key per thread, if any)
    uint32_t cap = dense ? 512u : final_cap(a.K);
    while (dense && cap < (uint32_t)a.K + kSelThreads) cap <<= 1;
    // keys, ids, and the query row + a row of zeros for a query that has to be rescored; or the histograms (and what is
    // collected from a range of values)
    const size_t hists = (size_t)4 * 256 * sizeof(uint32_t);
    const size_t qbytes = dense ? hists + survivors((uint32_t)a.K, a.width) * sizeof(u64) : std::max((size_t)2 * (a.row_bytes + kQPadBytes), hists);
    // ..., and the query's rows of the candidate layout
    const size_t lds = (size_t)cap * sizeof(u64) + (size_t)((a.k + 1) & ~1) * sizeof(int64_t) + qbytes +
                       (size_t)(4 * a.nprobe + 1) * sizeof(uint32_t);
    static LdsCleared cleared[2]; // (k and nprobe of some hundreds take more than 64 KB)
    const auto kernel = dense ? select_final_kernel<true> : select_final_kernel<false>;
    if (lds > 48 * 1024) {
        const hipError_t e = allow_lds(kernel, cleared[dense], 1024);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3((uint32_t)nq), dim3(kSelThreads), lds, s, a, h, cap, (uint32_t)qbytes);
    return hipGetLastError();
}

// ------------------------------------------------------------------ scope union

// Merge of the per-handle results of one query (Section 3.2: a request searches the memories
// of a set of agents and merges what each returns).  Every handle's row is already sorted
// (value, id); a candidate's key is (value key, position of the handle in the scope, rank
// inside that handle's row), so equal values come out by handle, then by id.
__global__ __launch_bounds__(kSelThreads) void union_merge_kernel(UnionArgs a)
{
    __shared__ u64 keys[kSelCap];
    __shared__ uint32_t s_cnt;
    const size_t q = blockIdx.x;
    const uint32_t k = (uint32_t)a.k, total = (uint32_t)a.n_handles * k;
    Selector sel;
    sel.init(keys, &s_cnt, a.k);
    for (uint32_t base = 0; base < total; base += kSelThreads) {
        sel.reserve(kSelThreads);
        const uint32_t i = base + threadIdx.x;
        if (i < total) {
            const uint32_t h = i / k, j = i - h * k;
            const size_t at = ((size_t)h * a.nq + q) * k + j;
            if (a.ids[at] >= 0) sel.push(((u64)order_bits(a.dist[at], a.metric) << 32) | (u64)(h << 10 | j));
        }
    }
    sel.flush();
    const uint32_t n = s_cnt;
    for (uint32_t j = threadIdx.x; j < k; j += kSelThreads) {
        const size_t o = q * k + j;
        if (j < n) {
            const uint32_t lo = (uint32_t)keys[j];
            const uint32_t h = (lo >> 10) & 0x7fu, r = lo & 0x3ffu;
            const size_t at = ((size_t)h * a.nq + q) * k + r;
            a.out_src[o] = (int32_t)h;
            a.out_ids[o] = a.ids[at];
            a.out_dist[o] = a.dist[at];
        } else {
            a.out_src[o] = -1;
            a.out_ids[o] = -1;
            a.out_dist[o] = a.metric == PK_METRIC_IP ? -INFINITY : INFINITY;
        }
    }
}

hipError_t launch_union_merge(const UnionArgs &a, hipStream_t s)
{
    if (a.nq <= 0) return hipSuccess;
    if (a.k < 1 || a.k > PK_MAX_K || a.n_handles < 1 || a.n_handles > PK_MAX_HANDLES) return hipErrorInvalidValue;
    hipLaunchKernelGGL(union_merge_kernel, dim3((uint32_t)a.nq), dim3(kSelThreads), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------ level cascade

// Section 4.2, early termination: one wave per query.  An open query takes this level's row;
// it ends here if the row holds k candidates and the k-th (the farthest of a row sorted best
// first) beats the query's threshold, or if this is the last level.
__global__ __launch_bounds__(256) void level_accept_kernel(LevelArgs a)
{
    const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (q >= a.nq) return;
    if (!a.first && a.open[q] == 0u) return;
    const size_t row = (size_t)q * a.k;
    if (a.row_ids) {
        for (int j = lane; j < a.k; j += 64) {
            a.out_ids[row + j] = a.row_ids[row + j];
            a.out_dist[row + j] = a.row_dist[row + j];
        }
    }
    if (lane == 0) {
        const int64_t *ids = a.row_ids ? a.row_ids : a.out_ids;
        const float *dist = a.row_ids ? a.row_dist : a.out_dist;
        const bool full = ids[row + a.k - 1] >= 0;
        const float kth = dist[row + a.k - 1], t = a.stop[q];
        const bool beats = a.metric == PK_METRIC_IP ? kth > t : kth < t;
        const bool done = a.last || (full && beats);
        a.open[q] = done ? 0u : 1u;
        if (a.level_out && (done || a.first)) a.level_out[q] = a.level;
    }
}

hipError_t launch_level_accept(const LevelArgs &a, hipStream_t s)
{
    if (a.nq <= 0) return hipSuccess;
    hipLaunchKernelGGL(level_accept_kernel, dim3((uint32_t)((a.nq + 3) / 4)), dim3(256), 0, s, a);
    return hipGetLastError();
}

__global__ void level_mask_kernel(int32_t *probes, int nprobe, const uint32_t *open, int64_t nq)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nq * nprobe) return;
    if (open[i / nprobe] == 0u) probes[i] = -1;
}

hipError_t launch_level_mask(int32_t *probes, int nprobe, const uint32_t *open, int64_t nq, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    const int64_t n = nq * nprobe;
    hipLaunchKernelGGL(level_mask_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, probes, nprobe, open, nq);
    return hipGetLastError();
}

} // namespace pk
