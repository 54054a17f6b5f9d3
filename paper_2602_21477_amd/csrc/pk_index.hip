// Index construction and the insert path (device side).
//
// Section 3.1 / Section 6.1 "IVF-Static": a vector is appended to the list of its nearest
// centroid and nothing else changes.  Section 4.4 keeps new vectors of a GPU-resident
// cluster in a CPU-side buffer because a device list cannot grow in place; here a list
// is a chain of fixed-size pages, so growing it means taking the next free page of the
// arena: no reallocation, no copy of old data, no host involvement.
#include <algorithm>

#include "pk_internal.h"

namespace pk {

// centroid table in scan layout: [nlist_pad][dpad32] fp32, zero padded, plus squared norms
__global__ __launch_bounds__(256) void store_centroids_kernel(const float *c, int nlist, int d, int dpad32, int metric,
                                                              float *cent, float *cnorm)
{
    __shared__ float s_part[4];
    const int row = blockIdx.x;
    float acc = 0.f;
    for (int i = threadIdx.x; i < dpad32; i += blockDim.x) {
        const float v = (row < nlist && i < d) ? c[(size_t)row * d + i] : 0.f;
        cent[(size_t)row * dpad32 + i] = v;
        acc += v * v;
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) cnorm[row] = metric == PK_METRIC_L2 ? s_part[0] + s_part[1] + s_part[2] + s_part[3] : 0.f;
}

hipError_t launch_store_centroids(const float *c, int nlist, int d, int dpad32, int nlist_pad, int metric, float *cent,
                                  float *cnorm, hipStream_t s)
{
    hipLaunchKernelGGL(store_centroids_kernel, dim3(nlist_pad), dim3(256), 0, s, c, nlist, d, dpad32, metric, cent,
                       cnorm);
    return hipGetLastError();
}

// One word per list serialises its atomics (262 144 rows over 162 lists: 187 us): a workgroup counts a run of rows in
// LDS first and adds each list's count once.  More lists than LDS takes spread the atomics by themselves.
__global__ __launch_bounds__(256) void lists_of_best_kernel(const unsigned long long *best, int64_t n, int nlist,
                                                            int32_t *assign, uint32_t *cnt, uint32_t *slots, int64_t run, bool lds)
{
    extern __shared__ uint32_t s_cnt[];
    if (lds) {
        for (int l = threadIdx.x; l < nlist; l += 256) s_cnt[l] = 0u;
        __syncthreads();
    }
    const int64_t i0 = (int64_t)blockIdx.x * run, i1 = i0 + run < n ? i0 + run : n;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
        const uint32_t l = (uint32_t)best[i];
        assign[i] = (int32_t)l;
        if (l >= (uint32_t)nlist) continue;
        const uint32_t at = atomicAdd(lds ? &s_cnt[l] : &cnt[l], 1u);
        if (slots) slots[i] = at;
    }
    if (!lds) return;
    __syncthreads();
    for (int l = threadIdx.x; l < nlist; l += 256)
        if (s_cnt[l]) s_cnt[l] = atomicAdd(&cnt[l], s_cnt[l]);
    if (!slots) return;
    __syncthreads();
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
        const uint32_t l = (uint32_t)best[i];
        if (l < (uint32_t)nlist) slots[i] += s_cnt[l]; // (the thread's own)
    }
}

hipError_t launch_lists_of_best(const unsigned long long *best, int64_t n, int nlist, int32_t *assign, uint32_t *cnt, uint32_t *slots, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const bool lds = nlist <= kLdsLists;
    int64_t run = 2048; // rows per workgroup: at most 1024 workgroups add their counts to the same words
    while ((n + run - 1) / run > 1024) run *= 2;
    hipLaunchKernelGGL(lists_of_best_kernel, dim3((uint32_t)((n + run - 1) / run)), dim3(256), lds ? (size_t)nlist * 4 : 0, s,
                       best, n, nlist, assign, cnt, slots, run, lds);
    return hipGetLastError();
}

// one wave writes one vector into slot `slot` of list `l`: convert (fp16: round to nearest
// even), zero pad the row, squared norm of the stored values, id
__device__ void write_row(const DevIndex &ix, uint32_t l, uint32_t slot, const float *src, int64_t id)
{
    const uint32_t P = (uint32_t)ix.P;
    const uint32_t lp = slot / P;
    const uint32_t pg = phys_page(ix, l, lp);
    const Arena &ar = arena_of(ix, pg);
    const size_t local = (size_t)(pg - ar.first_page) * P + (slot - lp * P);
    char *dst = ar.vec + local * (size_t)ix.row_bytes;
    const int lane = threadIdx.x & 63;
    const int n_el = ix.storage == PK_F16 ? ix.row_bytes / 2 : ix.row_bytes / 4;
    float acc = 0.f;
    constexpr int kBatch = 8; // elements read before the first of them is written: a load queues behind earlier stores
    for (int i0 = lane; i0 < n_el; i0 += 64 * kBatch) {
        float v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int i = i0 + 64 * u;
            v[u] = i < ix.d ? src[i] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int i = i0 + 64 * u;
            if (i >= n_el) continue;
            if (ix.storage == PK_F16) {
                const _Float16 h = (_Float16)v[u];
                reinterpret_cast<_Float16 *>(dst)[i] = h;
                v[u] = (float)h;
            } else {
                reinterpret_cast<float *>(dst)[i] = v[u];
            }
            acc += v[u] * v[u];
        }
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) {
        ar.norm[local] = acc;
        ar.ids[local] = id;
    }
}

// Build: the lists' extents from their lengths, one behind the other, and the pages they take together (ctr[0]; more than there
// are, ctr[2], and no row is placed).  One workgroup, 1024 lists at a time.
__global__ __launch_bounds__(1024) void build_pages_kernel(const DevIndex *ixp, const uint32_t *cnt)
{
    __shared__ uint32_t s_wave[16];
    const DevIndex &ix = *ixp;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, P = (uint32_t)ix.P, nlist = (uint32_t)ix.nlist;
    uint64_t before = 0; // pages of the lists before this round's
    for (uint32_t l0 = 0; l0 < nlist; l0 += 1024u) {
        const uint32_t l = l0 + tid, len = l < nlist ? cnt[l] : 0u, pages = (len + P - 1u) / P;
        uint32_t upto = pages; // of this thread's list and the wave's before it
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(upto, off);
            if (lane >= (uint32_t)off) upto += y;
        }
        if (lane == 63u) s_wave[wave] = upto;
        __syncthreads();
        uint32_t ahead = 0, all = 0;
        for (uint32_t w = 0; w < 16u; ++w) {
            ahead += w < wave ? s_wave[w] : 0u;
            all += s_wave[w];
        }
        if (l < nlist) {
            ix.main_base[l] = (uint32_t)before + ahead + upto - pages;
            ix.main_pages[l] = pages;
            ix.list_len[l] = len;
        }
        before += all;
        __syncthreads(); // (s_wave: read before the next round writes it)
    }
    if (tid == 0) ix.ctr[0] = before < 0xffffffffull ? (uint32_t)before : 0xffffffffu;
}

hipError_t launch_build_pages(const DevIndex *ix, const uint32_t *cnt, hipStream_t s)
{
    hipLaunchKernelGGL(build_pages_kernel, dim3(1), dim3(1024), 0, s, ix, cnt);
    return hipGetLastError();
}

// From a row's place in its list to its number among all rows of the build-time extents (fewer than 2^32 of at least 256 bytes
// fit the card), in place: what the scatter needs is then one word per row.  With list and place kept apart the scratch of
// 300 000 rows passes 2 MB, from where on mapping and unmapping it takes 0.6 ms (build of 300 000 x 1024 2514 and 1896 us).
constexpr uint32_t kNoRow = 0xffffffffu;
__global__ __launch_bounds__(256) void build_places_kernel(const DevIndex *ixp, const int32_t *assign, int64_t n, uint32_t *slots)
{
    const DevIndex &ix = *ixp;
    const bool fit = ix.ctr[0] <= ix.ctr[2];
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const uint32_t l = (uint32_t)assign[i]; // (no assignment leaves a number beyond the table, and it is not counted either)
        slots[i] = fit && l < (uint32_t)ix.nlist ? ix.main_base[l] * (uint32_t)ix.P + slots[i] : kNoRow;
    }
}

// Build: every vector into its slot of its list's build-time extent.  A wave takes `each` rows (at most 64): where a row
// goes is worked out by a lane of its own, all rows at once, and the rows are then copied eight 256-byte pieces at a time,
// whatever rows they belong to; a row's values are converted and summed as write_row does it.  Bound by memory: 300 000
// rows of 4 KB at 5.5 TB/s.  (A wave per row, its slot by an atomic of its own, waited for them row by row: 715 000 rows
// of 49 floats into 87 lists 1.93 ms.)
__global__ __launch_bounds__(256) void scatter_build_kernel(const DevIndex *ixp, const float *x, const int64_t *ids,
                                                            const uint32_t *rows_at, int64_t n, int64_t id0, int each)
{
    const DevIndex &ix = *ixp;
    const int lane = threadIdx.x & 63;
    const int64_t i0 = ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * each;
    if (i0 >= n) return;
    const int rows = (int)(n - i0 < each ? n - i0 : each);
    const uint32_t P = (uint32_t)ix.P;
    char *dst = nullptr;
    float *to_norm = nullptr;
    if (lane < rows) {
        const uint32_t at = rows_at[i0 + lane];
        if (at != kNoRow) {
            const uint32_t pg = at / P;
            const Arena &ar = arena_of(ix, pg);
            const size_t local = at - (size_t)ar.first_page * P;
            dst = ar.vec + local * (size_t)ix.row_bytes;
            to_norm = ar.norm + local;
            ar.ids[local] = ids ? ids[i0 + lane] : id0 + i0 + lane;
        }
    }
    const bool f16 = ix.storage == PK_F16;
    const int d = ix.d, n_el = f16 ? ix.row_bytes / 2 : ix.row_bytes / 4, pieces = n_el / 64; // (rows are whole 256 bytes)
    float acc = 0.f, norm = 0.f;
    int lr = 0, lc = 0, sr = 0, sc = 0; // row and piece of the next load and of the next store
    while (sr < rows) {
        constexpr int kBatch = 8; // pieces read before the first of them is written: a load queues behind earlier stores
        float v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int r = lr < rows ? lr : rows - 1, e = lc * 64 + lane;
            const float w = x[(size_t)(i0 + r) * d + (e < d ? e : d - 1)];
            v[u] = e < d ? w : 0.f;
            if (++lc == pieces) {
                lc = 0;
                ++lr;
            }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (sr >= rows) break;
            const uint64_t at = reinterpret_cast<uint64_t>(dst);
            char *const to = reinterpret_cast<char *>(((uint64_t)__builtin_amdgcn_readlane((uint32_t)(at >> 32), sr) << 32) |
                                                      (uint32_t)__builtin_amdgcn_readlane((uint32_t)at, sr));
            const int e = sc * 64 + lane;
            if (to) {
                if (f16) {
                    const _Float16 h = (_Float16)v[u];
                    reinterpret_cast<_Float16 *>(to)[e] = h;
                    v[u] = (float)h;
                } else {
                    reinterpret_cast<float *>(to)[e] = v[u];
                }
            }
            acc += v[u] * v[u];
            if (++sc == pieces) {
                for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
                norm = lane == sr ? acc : norm;
                acc = 0.f;
                sc = 0;
                ++sr;
            }
        }
    }
    if (to_norm) *to_norm = norm;
}

hipError_t launch_build_places(const DevIndex *ix, const int32_t *assign, int64_t n, uint32_t *slots, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int64_t want = (n + 255) / 256;
    hipLaunchKernelGGL(build_places_kernel, dim3((uint32_t)(want < 4096 ? want : 4096)), dim3(256), 0, s, ix, assign, n, slots);
    return hipGetLastError();
}

hipError_t launch_scatter_build(const DevIndex *ix, const float *x, const int64_t *ids, const uint32_t *rows_at, int64_t n, int64_t id0,
                                int pieces, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    // 64 pieces of 256 bytes per wave, 4 rows at least (with 32 rows of 4 KB the last of few rounds is nearly empty: 545 us), and
    // no more rows than leave every CU its 32 waves
    int each = std::max(4, std::min(64, 64 / std::max(pieces, 1)));
    while (each > 4 && n / each < 8192) each /= 2;
    hipLaunchKernelGGL(scatter_build_kernel, dim3((uint32_t)((n + 4 * each - 1) / (4 * each))), dim3(256), 0, s, ix, x, ids, rows_at, n, id0, each);
    return hipGetLastError();
}

// Insert, step 1b (batches of more than kFusedAppend vectors per handle): for every vector the number of earlier members of
// its group (kInsertGroup consecutive vectors of a handle) that go to the same list, and whether it is the group's
// last one (top bit).  A wave per vector over the group's lists: the same counts by one workgroup, a thread per
// vector, were 32 of the 38 us that reserving 1000 slots took.  Also turns the top-1 keys into lists (assign_out).
__global__ __launch_bounds__(256) void insert_rank_kernel(MultiArgs ma, const int32_t *assign, const unsigned long long *best,
                                                          const unsigned long long *redo, int32_t *assign_out, uint32_t *ranks)
{
    const uint32_t i = blockIdx.x * 4u + (threadIdx.x >> 6), lane = threadIdx.x & 63u;
    if (i >= ma.qlo[ma.n]) return;
    int h = 0;
    while (h + 1 < ma.n && i >= ma.qlo[h + 1]) ++h;
    const uint32_t row0 = ma.qlo[h], g0 = row0 + (i - row0) / kInsertGroup * kInsertGroup;
    const uint32_t g1 = g0 + kInsertGroup < ma.qlo[h + 1] ? g0 + kInsertGroup : ma.qlo[h + 1];
    auto list_of = [&](uint32_t j) { return best ? (int32_t)(uint32_t)best[j] : assign[j]; };
    auto open = [&](int32_t l) { return redo && l == kListByRedo; }; // (one of many)
    int32_t l = list_of(i);
    if (open(l)) l = (int32_t)(uint32_t)redo[i];
    uint32_t before = 0, after = 0;
    constexpr int U = 4; // requests in flight
    for (uint32_t j0 = g0 + lane; j0 < g1; j0 += 64u * U) {
        int32_t o[U];
#pragma unroll
        for (int u = 0; u < U; ++u) o[u] = j0 + 64u * u < g1 ? list_of(j0 + 64u * u) : -2;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t j = j0 + 64u * u;
            if (open(o[u])) o[u] = (int32_t)(uint32_t)redo[j];
            before += o[u] == l && j < i ? 1u : 0u;
            after += o[u] == l && j > i ? 1u : 0u;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        before += __shfl_xor(before, off);
        after += __shfl_xor(after, off);
    }
    if (lane == 0) {
        ranks[i] = before | (after == 0u ? 0x80000000u : 0u);
        if (best || redo) assign_out[i] = l;
    }
}

// Insert, step 2: slot reservation, one workgroup per handle, a group of at most kInsertGroup vectors after the other.
// Vector i takes slot list_len[l] + (number of earlier group members of the same list), so the order inside a list
// is the arrival order.  A vector whose slot starts a page beyond the build-time extent opens a delta page.  If the
// arena or a list's delta table cannot take the whole group, nothing of it is inserted, its slots are 0xffffffff and
// the sticky error flag is set.  Small batches (x given, no ranks): the workgroup's 16 waves also write the rows
// (step 3), which saves the launch that would otherwise follow.
template <bool RANKED>
__global__ __launch_bounds__(1024) void reserve_kernel(MultiArgs ma, const int32_t *assign, const uint32_t *ranks,
                                                       unsigned long long *best, uint32_t *slots, int32_t *assigned_out,
                                                       AppendIds idc, const float *x, const int64_t *ids)
{
    __shared__ int32_t s_l[1024];
    __shared__ uint32_t s_slot[1024];
    __shared__ uint32_t s_need, s_bad, s_page0;
    static_assert(kInsertGroup == 1024, "a thread per vector of a group");
    // workgroup a serves handle a: its vectors are rows [qlo[a], qlo[a+1]) of the batch
    const DevIndex &ix = *ma.ix[blockIdx.x];
    const uint32_t row0 = ma.qlo[blockIdx.x];
    const int m = (int)(ma.qlo[blockIdx.x + 1] - row0);
    if (m == 0) return;
    if (assign) assign += row0;
    if constexpr (RANKED) ranks += row0;
    slots += row0;
    if (assigned_out) assigned_out += row0;
    for (int g0 = 0; g0 < (RANKED ? m : 1); g0 += kInsertGroup) { // (without ranks: one group of at most kFusedAppend)
        const int t = threadIdx.x, i = g0 + t;
        if (t == 0) {
            s_need = 0;
            s_bad = 0;
        }
        int32_t l = -1;
        uint32_t rank = 0;
        bool last = false;
        if (i < m) {
            if (assign) {
                l = assign[i];
            } else { // the top-1 key the centroid kernel left (reset for the next insert on the way out)
                l = (int32_t)(uint32_t)best[row0 + i];
            }
            if (l < 0 || l >= ix.nlist) l = -1;
            if constexpr (RANKED) {
                rank = ranks[i] & 0x7fffffffu;
                last = (ranks[i] >> 31) != 0u;
            }
        }
        s_l[t] = l;
        __syncthreads();
        if (!RANKED && l >= 0) {
            uint32_t cnt = 0;
            for (int j = 0; j < m; ++j) {
                const bool same = s_l[j] == l;
                cnt += same ? 1u : 0u;
                rank += (same && j < i) ? 1u : 0u;
            }
            last = rank == cnt - 1;
        }
        uint32_t slot = 0xffffffffu, di = 0;
        bool opens = false;
        if (l >= 0) {
            slot = ix.list_len[l] + rank;
            const uint32_t lp = slot / (uint32_t)ix.P;
            if (slot % (uint32_t)ix.P == 0 && lp >= ix.main_pages[l]) {
                di = lp - ix.main_pages[l];
                if (di >= (uint32_t)ix.max_dp) atomicOr(&s_bad, (uint32_t)kErrListFull);
                // a list that shrank (deletes) still owns the delta pages it had: take a new one
                // only where the table has none
                else opens = ix.dtab[(size_t)l * ix.max_dp + di] == 0xffffffffu;
            }
        } else if (i < m) {
            atomicOr(&s_bad, (uint32_t)kErrListFull);
        }
        uint32_t my_page = 0;
        if (opens) my_page = atomicAdd(&s_need, 1u);
        __syncthreads();
        if (t == 0) {
            const uint32_t p0 = ix.ctr[0];
            s_page0 = p0;
            if (p0 + s_need > ix.ctr[2]) s_bad |= (uint32_t)kErrPages;
            if (s_bad) atomicOr(&ix.ctr[1], s_bad);
            else ix.ctr[0] = p0 + s_need;
        }
        __syncthreads();
        const bool ok = s_bad == 0;
        if (ok && opens) ix.dtab[(size_t)l * ix.max_dp + di] = s_page0 + my_page;
        if (ok && l >= 0 && last) ix.list_len[l] = slot + 1;
        if (i < m) {
            slots[i] = ok ? slot : 0xffffffffu;
            if (assigned_out) assigned_out[i] = l;
        }
        s_slot[t] = ok ? slot : 0xffffffffu;
        __syncthreads(); // slots, and the page table entries and lengths just written, are visible to the whole workgroup
    }
    if constexpr (RANKED) return;
    for (int r = (int)threadIdx.x >> 6; r < m; r += 16) {
        if (s_slot[r] == 0xffffffffu) continue;
        const uint32_t row = row0 + (uint32_t)r;
        write_row(ix, (uint32_t)s_l[r], s_slot[r], x + (size_t)row * ix.d,
                  ids ? ids[row] : idc.id0[blockIdx.x] + (int64_t)r);
    }
    if (best && !assign && (int)threadIdx.x < m) best[row0 + threadIdx.x] = ~0ull;
}

hipError_t launch_reserve(const MultiArgs &ma, const int32_t *assign, const unsigned long long *best,
                          const unsigned long long *redo, int32_t *lists, uint32_t *ranks, uint32_t *slots, int32_t *assigned_out, hipStream_t s)
{
    if (ma.n <= 0 || ma.qlo[ma.n] == 0) return hipSuccess;
    if ((assign == nullptr) == (best == nullptr) || !ranks || (best && !lists) || (redo && assign != lists)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(insert_rank_kernel, dim3((ma.qlo[ma.n] + 3) / 4), dim3(256), 0, s, ma, assign, best, redo, lists, ranks);
    hipLaunchKernelGGL(reserve_kernel<true>, dim3(ma.n), dim3(1024), 0, s, ma, best ? lists : assign, ranks, nullptr, slots, assigned_out,
                       AppendIds{}, nullptr, nullptr);
    return hipGetLastError();
}

// steps 2 and 3 in one launch, for batches of at most kFusedAppend vectors per handle
hipError_t launch_reserve_append(const MultiArgs &ma, const AppendIds &idc, const float *x, const int64_t *ids,
                                 const int32_t *assign, unsigned long long *best, uint32_t *slots, int32_t *assigned_out,
                                 hipStream_t s)
{
    if (ma.n <= 0 || ma.qlo[ma.n] == 0) return hipSuccess;
    if (!x || (!assign && !best)) return hipErrorInvalidValue;
    for (int a = 0; a < ma.n; ++a)
        if (ma.qlo[a + 1] - ma.qlo[a] > (uint32_t)kFusedAppend) return hipErrorInvalidValue;
    hipLaunchKernelGGL(reserve_kernel<false>, dim3(ma.n), dim3(1024), 0, s, ma, assign, nullptr, best, slots, assigned_out, idc, x, ids);
    return hipGetLastError();
}

// Insert, step 3: write the vectors into their reserved slots
// (reset: top-1 keys to put back to "none yet" for the next insert, or null)
__global__ __launch_bounds__(256) void append_kernel(MultiArgs ma, AppendIds idc, const float *x, const int64_t *ids,
                                                     const int32_t *assign, const uint32_t *slots, unsigned long long *reset)
{
    const int wave = threadIdx.x >> 6;
    const uint32_t i = blockIdx.x * 4 + wave;
    if (i >= ma.qlo[ma.n]) return;
    if (reset && (threadIdx.x & 63) == 0) reset[i] = ~0ull;
    int h = 0;
    while (h + 1 < ma.n && i >= ma.qlo[h + 1]) ++h;
    const DevIndex &ix = *ma.ix[h];
    const uint32_t slot = slots[i];
    if (slot == 0xffffffffu) return;
    write_row(ix, (uint32_t)assign[i], slot, x + (size_t)i * ix.d, ids ? ids[i] : idc.id0[h] + (int64_t)(i - ma.qlo[h]));
}

hipError_t launch_append(const MultiArgs &ma, const AppendIds &idc, const float *x, const int64_t *ids,
                         const int32_t *assign, const uint32_t *slots, unsigned long long *reset, hipStream_t s)
{
    const uint32_t m = ma.n > 0 ? ma.qlo[ma.n] : 0u;
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(append_kernel, dim3((m + 3) / 4), dim3(256), 0, s, ma, idc, x, ids, assign, slots, reset);
    return hipGetLastError();
}

// probes[:, 0] of a top-1 coarse search -> assignment array (stride nprobe = 1 is the identity;
// kept as a kernel so the copy stays on the stream)
// ------------------------------------------------------------------ delete

// location of position `pos` of list l: arena and row number inside the arena
__device__ __forceinline__ const Arena &locate(const DevIndex &ix, uint32_t l, uint32_t pos, size_t &local)
{
    const uint32_t P = (uint32_t)ix.P, lp = pos / P;
    const uint32_t pg = phys_page(ix, l, lp);
    const Arena &ar = arena_of(ix, pg);
    local = (size_t)(pg - ar.first_page) * P + (pos - lp * P);
    return ar;
}

// Deleting by id (Section 5's interface: delete, and update as delete + insert) in three launches, every one of them
// parallel over what it works on, so that a list of 400 000 rows costs what its share of the index's rows costs and
// no workgroup sorts anything (two sorts of 2000 keys by one workgroup each took 66 us):
//   find     every workgroup builds a hash set of the ids in LDS and looks its units of kDeleteUnit rows up in it; the
//            rows to go are noted as (list, position) in no order
//   rank     a wave per noted row counts its list's other noted rows, and those before it; the first of a list
//            shortens the list
//   move     a list that loses c rows keeps its first len - c positions: the rows to go among them are holes, and as
//            many rows beyond them stay; the i-th row that stays fills the i-th hole.  A wave per noted row finds its
//            move (row number t of the list's noted rows looks at position len - c + t) by counting, and makes it.
//            Every move reads and writes rows no other move touches, so they all run at once.
// Lists are unordered sets: no tombstones, nothing for the scan to skip.  The pages a list no longer
// reaches stay its own for later inserts.
// All launches of a call (fills and copies of the earlier sequence included): 8 ids among 1 M rows 54 -> 23 us, 2000 ids
// among 300 000 rows 113 -> 39; the calls, with their wait on the host, 89 -> 34 us and 265 -> 71 (no more than 27 where nobody carries the ids).

constexpr unsigned long long kNoId = 0x8000000000000000ull; // marks a free slot of the hash set (the id of that value is kept apart)

// units of the lists before each one, for tables longer than a workgroup takes along
__global__ __launch_bounds__(1024) void delete_units_kernel(DeleteArgs a)
{
    __shared__ uint32_t s_wave[17];
    const DevIndex &ix = *a.ix;
    for (int l = threadIdx.x; l < a.nlist; l += blockDim.x) a.unit_start[l] = (ix.list_len[l] + kDeleteUnit - 1) / kDeleteUnit;
    __syncthreads();
    const uint32_t units = block_exscan(a.unit_start, a.unit_start, (uint32_t)a.nlist, s_wave);
    if (threadIdx.x == 0) a.unit_start[a.nlist] = units;
}

// dynamic LDS (all of the kernel's: the limit set for it counts static LDS in): kFindHead words, the hash set
// [1 << a.bits], then (if in_lds) the units of the lists before each one
constexpr int kFindHead = 24;
__global__ __launch_bounds__(256) void delete_find_kernel(DeleteArgs a, bool in_lds)
{
    extern __shared__ __align__(16) uint32_t s_head[];
    uint32_t *s_wave = s_head;          // [17]
    uint32_t &s_has = s_head[20];       // the id that the free mark stands for is among the ids
    unsigned long long *s_set = reinterpret_cast<unsigned long long *>(s_head + kFindHead);
    const DevIndex &ix = *a.ix;
    const uint32_t mask = (1u << a.bits) - 1u;
    uint32_t *s_unit = reinterpret_cast<uint32_t *>(s_set + mask + 1);
    auto slot_of = [&](unsigned long long id) { return (uint32_t)((id * 0x9E3779B97F4A7C15ull) >> (64 - a.bits)); };
    uint32_t units;
    const uint32_t *start = in_lds ? s_unit : a.unit_start;
    const uint32_t *list_len = ix.list_len;
    constexpr int B = 8; // ids requested before the first of them goes into the set
    const long long *ids = reinterpret_cast<const long long *>(a.ids);
    unsigned long long mine[B];
#pragma unroll
    for (int u = 0; u < B; ++u) mine[u] = (int)threadIdx.x + 256 * u < a.m ? (unsigned long long)ids[threadIdx.x + 256 * u] : kNoId;
    if (in_lds) {
        for (int l0 = threadIdx.x; l0 < a.nlist; l0 += 256 * B) {
            uint32_t len[B];
#pragma unroll
            for (int u = 0; u < B; ++u) len[u] = l0 + 256 * u < a.nlist ? list_len[l0 + 256 * u] : 0u;
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (l0 + 256 * u < a.nlist) s_unit[l0 + 256 * u] = (len[u] + kDeleteUnit - 1) / kDeleteUnit;
        }
        __syncthreads();
        units = block_exscan(s_unit, s_unit, (uint32_t)a.nlist, s_wave);
    } else {
        units = a.unit_start[a.nlist];
    }
    if (blockIdx.x >= units) return; // nothing to look up
    for (uint32_t i = threadIdx.x; i <= mask; i += 256) s_set[i] = kNoId;
    if (threadIdx.x == 0) s_has = 0;
    __syncthreads();
    for (int i0 = threadIdx.x; i0 < a.m; i0 += 256 * B) {
        if (i0 >= 256 * B) {
#pragma unroll
            for (int u = 0; u < B; ++u) mine[u] = i0 + 256 * u < a.m ? (unsigned long long)ids[i0 + 256 * u] : kNoId;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if (i0 + 256 * u >= a.m) continue;
            const unsigned long long id = mine[u];
            if (id == kNoId) {
                s_has = 1;
                continue;
            }
            uint32_t at = slot_of(id); // the set is at most half full: a free slot or the id itself comes up
            while (true) {
                const unsigned long long was = atomicCAS(&s_set[at], kNoId, id);
                if (was == kNoId || was == id) break;
                at = (at + 1u) & mask;
            }
        }
    }
    __syncthreads();
    const bool has = s_has != 0;
    for (uint32_t u = blockIdx.x; u < units; u += gridDim.x) {
        uint32_t lo = 0, hi = (uint32_t)a.nlist - 1; // the last list whose units start at or before u
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (start[mid] <= u) lo = mid;
            else hi = mid - 1;
        }
        const uint32_t l = lo, len = list_len[l], P = (uint32_t)ix.P, mp = ix.main_pages[l], mb = ix.main_base[l];
        const uint32_t base = (u - start[l]) * (uint32_t)kDeleteUnit;
        constexpr int R = kDeleteUnit / 256;
        unsigned long long id[R];
#pragma unroll
        for (int j = 0; j < R; ++j) { // all requested before the first is looked up
            const uint32_t pos = base + (uint32_t)j * 256u + threadIdx.x;
            id[j] = 0;
            if (pos >= len) continue;
            const uint32_t lp = pos / P;
            const uint32_t pg = lp < mp ? mb + lp : ix.dtab[(size_t)l * ix.max_dp + (lp - mp)];
            const Arena &ar = arena_of(ix, pg);
            id[j] = (unsigned long long)ar.ids[(size_t)(pg - ar.first_page) * P + (pos - lp * P)];
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const uint32_t pos = base + (uint32_t)j * 256u + threadIdx.x;
            if (pos >= len) continue;
            bool hit = has && id[j] == kNoId;
            if (id[j] != kNoId)
                for (uint32_t at = slot_of(id[j]); s_set[at] != kNoId; at = (at + 1u) & mask)
                    if (s_set[at] == id[j]) {
                        hit = true;
                        break;
                    }
            if (hit) {
                const uint32_t at = atomicAdd(&a.scal[0], 1u);
                if (at < (uint32_t)kDeleteChunk) a.hits[at] = ((unsigned long long)l << 32) | pos;
            }
        }
    }
}

__global__ __launch_bounds__(256) void delete_rank_kernel(DeleteArgs a)
{
    __shared__ unsigned long long s_hits[kDeleteChunk];
    const DevIndex &ix = *a.ix;
    const uint32_t found = a.scal[0];
    const uint32_t nh = found < (uint32_t)kDeleteChunk ? found : (uint32_t)kDeleteChunk;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.scal[1] = nh; // what the move kernel goes by
        const unsigned long long removed = (a.first ? 0ull : *a.removed) + nh;
        const uint32_t again = (a.first ? 0u : a.scal[2]) | (found > nh ? 1u : 0u); // more rows carried the ids than a pass takes
        *a.removed = removed;
        a.scal[2] = again;
        // for the host, which reads them once the stream is idle
        __hip_atomic_store(a.host, (uint32_t)removed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(a.host + 1, (uint32_t)(removed >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(a.host + 2, again, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (blockIdx.x * 4u >= nh) return;
    for (uint32_t i = threadIdx.x; i < nh; i += 256) s_hits[i] = a.hits[i];
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t g = blockIdx.x * 4u + (threadIdx.x >> 6); g < nh; g += gridDim.x * 4u) {
        const unsigned long long key = s_hits[g];
        const uint32_t l = (uint32_t)(key >> 32);
        uint32_t before = 0, all = 0;
        for (uint32_t j = lane; j < nh; j += 64) {
            const unsigned long long o = s_hits[j];
            all += (uint32_t)(o >> 32) == l ? 1u : 0u;
            before += (uint32_t)(o >> 32) == l && o < key ? 1u : 0u;
        }
        for (int off = 32; off > 0; off >>= 1) {
            before += __shfl_xor(before, off);
            all += __shfl_xor(all, off);
        }
        if (lane == 0) {
            a.hit_rank[g] = before;
            a.hit_cnt[g] = all;
            if (before == 0) { // the only one of its list to look at the list's length
                const uint32_t len = ix.list_len[l];
                a.hit_len0[g] = len;
                ix.list_len[l] = len - all;
            }
        }
    }
}

__global__ __launch_bounds__(256) void delete_move_kernel(DeleteArgs a)
{
    __shared__ unsigned long long s_hits[kDeleteChunk];
    __shared__ uint16_t s_rank[kDeleteChunk];
    const DevIndex &ix = *a.ix;
    const uint32_t nh = a.scal[1];
    if (blockIdx.x == 0 && threadIdx.x == 0) a.scal[0] = 0; // for the next call (nothing else of this launch reads it)
    if (blockIdx.x * 4u >= nh) return;
    for (uint32_t i = threadIdx.x; i < nh; i += 256) {
        s_hits[i] = a.hits[i];
        s_rank[i] = (uint16_t)a.hit_rank[i];
    }
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t g = blockIdx.x * 4u + (threadIdx.x >> 6); g < nh; g += gridDim.x * 4u) {
        const uint32_t l = (uint32_t)(s_hits[g] >> 32), t = s_rank[g], c = a.hit_cnt[g];
        // the list's first noted row knows how long the list was
        uint32_t first = 0xffffffffu;
        for (uint32_t j = lane; j < nh; j += 64)
            if ((uint32_t)(s_hits[j] >> 32) == l && s_rank[j] == 0) first = j;
        for (int off = 32; off > 0; off >>= 1) first = min(first, (uint32_t)__shfl_xor(first, off));
        const uint32_t newlen = a.hit_len0[first] - c, p = newlen + t; // position number t of the c beyond the new end
        uint32_t holes = 0, below = 0, goes = 0; // rows to go among the positions that stay; before p; at p
        for (uint32_t j = lane; j < nh; j += 64) {
            const unsigned long long o = s_hits[j];
            if ((uint32_t)(o >> 32) != l) continue;
            const uint32_t pos = (uint32_t)o;
            holes += pos < newlen ? 1u : 0u;
            below += pos < p ? 1u : 0u;
            goes += pos == p ? 1u : 0u;
        }
        for (int off = 32; off > 0; off >>= 1) {
            holes += __shfl_xor(holes, off);
            below += __shfl_xor(below, off);
            goes += __shfl_xor(goes, off);
        }
        if (goes) continue; // (wave-uniform)
        // the row stays: it is number i of those that do, and fills the list's i-th hole
        const uint32_t i = t - (below - holes);
        uint32_t dst_pos = 0xffffffffu;
        for (uint32_t j = lane; j < nh; j += 64)
            if ((uint32_t)(s_hits[j] >> 32) == l && s_rank[j] == i) dst_pos = (uint32_t)s_hits[j];
        for (int off = 32; off > 0; off >>= 1) dst_pos = min(dst_pos, (uint32_t)__shfl_xor(dst_pos, off));
        size_t ls, ld;
        const Arena &as = locate(ix, l, p, ls);
        const Arena &ad = locate(ix, l, dst_pos, ld);
        const int row_bytes = ix.row_bytes;
        const uint4 *src = reinterpret_cast<const uint4 *>(as.vec + ls * (size_t)row_bytes);
        uint4 *dst = reinterpret_cast<uint4 *>(ad.vec + ld * (size_t)row_bytes);
        for (int w = (int)lane; w < row_bytes / 16; w += 64) dst[w] = src[w];
        if (lane == 0) {
            ad.norm[ld] = as.norm[ls];
            ad.ids[ld] = as.ids[ls];
        }
    }
}

hipError_t launch_delete(DeleteArgs a, int num_cu, hipStream_t s)
{
    if (a.m <= 0) return hipSuccess;
    if (a.m > kDeleteChunk || a.nlist < 1) return hipErrorInvalidValue;
    a.bits = 6;
    while ((1 << a.bits) < 2 * a.m) ++a.bits;
    const bool in_lds = a.nlist <= kLdsLists;
    if (!in_lds) hipLaunchKernelGGL(delete_units_kernel, dim3(1), dim3(1024), 0, s, a);
    const int lds = kFindHead * 4 + (int)((size_t)8 << a.bits) + (in_lds ? a.nlist * 4 : 0);
    static LdsCleared cleared;
    const hipError_t e = allow_lds(&delete_find_kernel, cleared);
    if (e != hipSuccess) return e;
    const int per_cu = std::max(1, std::min(8, 160 * 1024 / lds));
    hipLaunchKernelGGL(delete_find_kernel, dim3(num_cu * per_cu), dim3(256), lds, s, a, in_lds);
    const int grid = std::min((a.m + 3) / 4, 512); // a wave per noted row (more rows than ids: the waves go round again)
    hipLaunchKernelGGL(delete_rank_kernel, dim3(grid), dim3(256), 0, s, a);
    hipLaunchKernelGGL(delete_move_kernel, dim3(grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------ compaction

// One workgroup per page of the new layout: page pg belongs to the list whose new extent
// contains it; its rows, norms and ids are copied from wherever the old layout keeps that
// logical page (build-time extent or delta page, any arena).  Positions inside a list do
// not change.
__global__ __launch_bounds__(256) void compact_pages_kernel(const DevIndex *srcp, const DevIndex *dstp,
                                                            const uint8_t *skip)
{
    __shared__ uint32_t s_list;
    const DevIndex &src = *srcp, &dst = *dstp;
    const uint32_t pg = blockIdx.x;
    if (threadIdx.x == 0) {
        // last list whose extent starts at or before pg (extents are in list order; a list
        // without pages shares its start with the next one and can never be the answer)
        uint32_t lo = 0, hi = (uint32_t)dst.nlist;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) / 2;
            if (dst.main_base[mid] <= pg) lo = mid;
            else hi = mid;
        }
        s_list = lo;
    }
    __syncthreads();
    const uint32_t l = s_list;
    // lists the caller fills itself (split lists and the lists they give rise to)
    if (l >= (uint32_t)src.nlist || (skip && skip[l])) return;
    const uint32_t lp = pg - dst.main_base[l];
    const uint32_t P = (uint32_t)dst.P;
    const uint32_t len = dst.list_len[l];
    if (lp >= dst.main_pages[l] || lp * P >= len) return;
    const uint32_t nrows = len - lp * P < P ? len - lp * P : P;
    const uint32_t opg = phys_page(src, l, lp);
    const Arena &sa = arena_of(src, opg), &da = arena_of(dst, pg);
    const size_t so = opg - sa.first_page, dn = pg - da.first_page;
    const int row_bytes = dst.row_bytes;
    const uint4 *sv = reinterpret_cast<const uint4 *>(sa.vec + so * P * (size_t)row_bytes);
    uint4 *dv = reinterpret_cast<uint4 *>(da.vec + dn * P * (size_t)row_bytes);
    const size_t nvec = (size_t)nrows * row_bytes / 16;
    for (size_t i = threadIdx.x; i < nvec; i += blockDim.x) dv[i] = sv[i];
    for (uint32_t i = threadIdx.x; i < nrows; i += blockDim.x) {
        da.norm[dn * P + i] = sa.norm[so * P + i];
        da.ids[dn * P + i] = sa.ids[so * P + i];
    }
}

hipError_t launch_compact_pages(const DevIndex *src, const DevIndex *dst, uint32_t new_pages, const uint8_t *skip,
                                hipStream_t s)
{
    if (new_pages == 0) return hipSuccess;
    hipLaunchKernelGGL(compact_pages_kernel, dim3(new_pages), dim3(256), 0, s, src, dst, skip);
    return hipGetLastError();
}

// ------------------------------------------------------------------ list read-back and split

// one wave per member of list l: the stored row as fp32 [d] (rows may be NULL) and its id (ids may be NULL)
__global__ __launch_bounds__(256) void gather_list_kernel(const DevIndex *ixp, uint32_t l, uint32_t limit, float *rows,
                                                          int64_t *ids)
{
    const DevIndex &ix = *ixp;
    const uint32_t r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= ix.list_len[l] || r >= limit) return;
    size_t local;
    const Arena &ar = locate(ix, l, r, local);
    const int lane = threadIdx.x & 63;
    if (rows) {
        const char *src = ar.vec + local * (size_t)ix.row_bytes;
        for (int i = lane; i < ix.d; i += 64)
            rows[(size_t)r * ix.d + i] = ix.storage == PK_F16 ? (float)reinterpret_cast<const _Float16 *>(src)[i]
                                                               : reinterpret_cast<const float *>(src)[i];
    }
    if (ids && lane == 0) ids[r] = ar.ids[local];
}

hipError_t launch_gather_list(const DevIndex *ix, uint32_t l, uint32_t len, float *rows, int64_t *ids, hipStream_t s)
{
    if (len == 0) return hipSuccess;
    hipLaunchKernelGGL(gather_list_kernel, dim3((len + 3) / 4), dim3(256), 0, s, ix, l, len, rows, ids);
    return hipGetLastError();
}

// ---- 2-means of the lists to split

// stored row -> element i as fp32
__device__ __forceinline__ float row_element(const char *row, int storage, int i)
{
    return storage == PK_F16 ? (float)reinterpret_cast<const _Float16 *>(row)[i] : reinterpret_cast<const float *>(row)[i];
}

// one workgroup per job: the members with the smallest and the largest id become the first centroids
__global__ __launch_bounds__(1024) void split_init_kernel(SplitArgs a)
{
    __shared__ long long s_id[2][16];
    __shared__ uint32_t s_pos[2][16];
    const DevIndex &ix = *a.ix;
    const uint32_t j = blockIdx.x, l = a.job_list[j], len = a.job_len[j];
    long long lo_id = INT64_MAX, hi_id = INT64_MIN;
    uint32_t lo_pos = 0xffffffffu, hi_pos = 0xffffffffu;
    for (uint32_t r = threadIdx.x; r < len; r += blockDim.x) {
        size_t local;
        const Arena &ar = locate(ix, l, r, local);
        const long long id = ar.ids[local];
        if (id < lo_id || (id == lo_id && r < lo_pos)) {
            lo_id = id;
            lo_pos = r;
        }
        if (id > hi_id || (id == hi_id && r < hi_pos)) {
            hi_id = id;
            hi_pos = r;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const long long oi = __shfl_xor(lo_id, off), pi = __shfl_xor(hi_id, off);
        const uint32_t op = __shfl_xor(lo_pos, off), pp = __shfl_xor(hi_pos, off);
        if (oi < lo_id || (oi == lo_id && op < lo_pos)) {
            lo_id = oi;
            lo_pos = op;
        }
        if (pi > hi_id || (pi == hi_id && pp < hi_pos)) {
            hi_id = pi;
            hi_pos = pp;
        }
    }
    if ((threadIdx.x & 63) == 0) {
        s_id[0][threadIdx.x >> 6] = lo_id;
        s_pos[0][threadIdx.x >> 6] = lo_pos;
        s_id[1][threadIdx.x >> 6] = hi_id;
        s_pos[1][threadIdx.x >> 6] = hi_pos;
    }
    __syncthreads();
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) { // every thread folds the waves' results the same way
        if (s_id[0][w] < lo_id || (s_id[0][w] == lo_id && s_pos[0][w] < lo_pos)) {
            lo_id = s_id[0][w];
            lo_pos = s_pos[0][w];
        }
        if (s_id[1][w] > hi_id || (s_id[1][w] == hi_id && s_pos[1][w] < hi_pos)) {
            hi_id = s_id[1][w];
            hi_pos = s_pos[1][w];
        }
    }
    const int d = ix.d;
    for (int side = 0; side < 2; ++side) {
        size_t local;
        const Arena &ar = locate(ix, l, side ? hi_pos : lo_pos, local);
        const char *row = ar.vec + local * (size_t)ix.row_bytes;
        for (int i = threadIdx.x; i < d; i += blockDim.x) {
            a.cent[((size_t)j * 2 + side) * d + i] = (double)row_element(row, ix.storage, i);
            a.sum[((size_t)j * 2 + side) * d + i] = 0.0;
        }
    }
    if (threadIdx.x < 2) a.cnt[(size_t)j * 2 + threadIdx.x] = 0ull;
}

// One workgroup per unit of kSplitUnit members of one job; a wave takes a quarter of them, row by row:
// the lanes share the row's elements, the two squared distances are reduced over the wave (fp32), and the
// row is added to the wave's running sum of its side.  The four waves' sums meet in LDS and go to the
// job's sums as one fp64 atomic per element and unit.
constexpr int kSplitEl = (PK_MAX_DIM + 63) / 64; // elements of a row per lane
__global__ __launch_bounds__(256) void split_assign_kernel(SplitArgs a)
{
    extern __shared__ __align__(16) float s_split[]; // [2][d] centroids, then [4][2][d] the waves' sums
    __shared__ uint32_t s_ones[4];
    const DevIndex &ix = *a.ix;
    const int d = ix.d, storage = ix.storage, row_bytes = ix.row_bytes;
    const uint32_t P = (uint32_t)ix.P;
    uint32_t lo = 0, hi = (uint32_t)a.njobs - 1; // the job this unit belongs to
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (a.job_unit0[mid] <= blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const uint32_t j = lo, l = a.job_list[j], len = a.job_len[j];
    const uint32_t first = (blockIdx.x - a.job_unit0[j]) * (uint32_t)kSplitUnit;
    float *s_c = s_split, *s_sum = s_split + 2 * d;
    for (int i = threadIdx.x; i < 2 * d; i += blockDim.x) s_c[i] = (float)a.cent[(size_t)j * 2 * d + i];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float c0[kSplitEl], c1[kSplitEl], acc0[kSplitEl], acc1[kSplitEl];
#pragma unroll
    for (int e = 0; e < kSplitEl; ++e) {
        const int i = lane + 64 * e;
        c0[e] = i < d ? s_c[i] : 0.f;
        c1[e] = i < d ? s_c[d + i] : 0.f;
        acc0[e] = acc1[e] = 0.f;
    }
    uint32_t ones = 0;
    const uint32_t r0 = first + (uint32_t)wave * (kSplitUnit / 4);
    const uint32_t r1 = min(r0 + (uint32_t)(kSplitUnit / 4), len);
    for (uint32_t r = r0; r < r1;) {
        // the rows of one page are neighbours in memory
        const uint32_t lp = r / P, in_page = r - lp * P;
        const uint32_t pg = phys_page(ix, l, lp);
        const Arena &ar = arena_of(ix, pg);
        const char *page = ar.vec + ((size_t)(pg - ar.first_page) * P) * (size_t)row_bytes;
        const uint32_t n = min(P - in_page, r1 - r);
        for (uint32_t t = 0; t < n; ++t) {
            const char *row = page + (size_t)(in_page + t) * row_bytes;
            float x[kSplitEl], s0 = 0.f, s1 = 0.f;
#pragma unroll
            for (int e = 0; e < kSplitEl; ++e) {
                const int i = lane + 64 * e;
                x[e] = i < d ? row_element(row, storage, i) : 0.f;
            }
#pragma unroll
            for (int e = 0; e < kSplitEl; ++e) {
                const float u0 = x[e] - c0[e], u1 = x[e] - c1[e];
                s0 += u0 * u0;
                s1 += u1 * u1;
            }
            for (int off = 32; off > 0; off >>= 1) {
                s0 += __shfl_xor(s0, off);
                s1 += __shfl_xor(s1, off);
            }
            const bool second = s1 < s0; // the same in every lane
            if (second) {
#pragma unroll
                for (int e = 0; e < kSplitEl; ++e) acc1[e] += x[e];
                ++ones;
            } else {
#pragma unroll
                for (int e = 0; e < kSplitEl; ++e) acc0[e] += x[e];
            }
            if (lane == 0) a.side[(size_t)a.job_row0[j] + r + t] = second ? 1 : 0;
        }
        r += n;
    }
#pragma unroll
    for (int e = 0; e < kSplitEl; ++e) {
        const int i = lane + 64 * e;
        if (i < d) {
            s_sum[((size_t)wave * 2 + 0) * d + i] = acc0[e];
            s_sum[((size_t)wave * 2 + 1) * d + i] = acc1[e];
        }
    }
    if (lane == 0) s_ones[wave] = ones;
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * d; i += blockDim.x) {
        const double v = ((double)s_sum[i] + (double)s_sum[2 * d + i]) + ((double)s_sum[4 * d + i] + (double)s_sum[6 * d + i]);
        if (v != 0.0) atomicAdd(&a.sum[(size_t)j * 2 * d + i], v);
    }
    if (threadIdx.x == 0) {
        const uint32_t rows = first < len ? min((uint32_t)kSplitUnit, len - first) : 0u;
        const uint32_t n1 = s_ones[0] + s_ones[1] + s_ones[2] + s_ones[3];
        if (rows - n1) atomicAdd(&a.cnt[(size_t)j * 2], (unsigned long long)(rows - n1));
        if (n1) atomicAdd(&a.cnt[(size_t)j * 2 + 1], (unsigned long long)n1);
    }
}

// one workgroup per job: centroids to the means of their members; sums and counts back to zero
__global__ __launch_bounds__(256) void split_update_kernel(SplitArgs a)
{
    const uint32_t j = blockIdx.x;
    const int d = a.ix->d;
    const unsigned long long n0 = a.cnt[(size_t)j * 2], n1 = a.cnt[(size_t)j * 2 + 1];
    for (int i = threadIdx.x; i < 2 * d; i += blockDim.x) {
        const unsigned long long n = i < d ? n0 : n1;
        const size_t at = (size_t)j * 2 * d + i;
        if (n > 0) a.cent[at] = a.sum[at] / (double)n;
        a.sum[at] = 0.0;
    }
    __syncthreads(); // every thread has read the counts
    if (threadIdx.x < 2) {
        a.cnt_out[(size_t)j * 2 + threadIdx.x] = threadIdx.x ? n1 : n0;
        a.cnt[(size_t)j * 2 + threadIdx.x] = 0ull;
    }
}

__global__ __launch_bounds__(256) void split_centroids_kernel(SplitArgs a, int nlist0, float *dense)
{
    const uint32_t j = blockIdx.x;
    const int d = a.ix->d;
    for (int i = threadIdx.x; i < d; i += blockDim.x) {
        dense[(size_t)a.job_list[j] * d + i] = (float)a.cent[(size_t)j * 2 * d + i];
        dense[(size_t)(nlist0 + j) * d + i] = (float)a.cent[((size_t)j * 2 + 1) * d + i];
    }
}

hipError_t launch_split_init(const SplitArgs &a, hipStream_t s)
{
    if (a.njobs <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_init_kernel, dim3(a.njobs), dim3(1024), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_split_iterate(const SplitArgs &a, uint32_t total_units, int d, hipStream_t s)
{
    if (a.njobs <= 0 || total_units == 0) return hipSuccess;
    if (d > PK_MAX_DIM) return hipErrorInvalidValue;
    const size_t lds = (size_t)10 * d * sizeof(float); // at most 60 KB
    hipLaunchKernelGGL(split_assign_kernel, dim3(total_units), dim3(256), lds, s, a);
    hipLaunchKernelGGL(split_update_kernel, dim3(a.njobs), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_split_centroids(const SplitArgs &a, int nlist0, float *dense, hipStream_t s)
{
    if (a.njobs <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_centroids_kernel, dim3(a.njobs), dim3(256), 0, s, a, nlist0, dense);
    return hipGetLastError();
}

// Stable partition of a list by side[r] in {0, 1}: slot[r] = number of earlier members on the
// same side (one workgroup walks the list)
__global__ __launch_bounds__(1024) void split_slots_kernel(const int32_t *side, uint32_t len, uint32_t *slot)
{
    __shared__ uint32_t s_wave[17];
    __shared__ uint32_t s_in[1024], s_out[1024];
    uint32_t ones = 0;
    for (uint32_t base = 0; base < len; base += 1024) {
        const uint32_t r = base + threadIdx.x;
        const uint32_t b = r < len && side[r] != 0 ? 1u : 0u;
        s_in[threadIdx.x] = b;
        __syncthreads();
        const uint32_t n = len - base < 1024u ? len - base : 1024u;
        const uint32_t total = block_exscan(s_in, s_out, n, s_wave);
        if (r < len) slot[r] = b ? ones + s_out[threadIdx.x] : r - (ones + s_out[threadIdx.x]);
        ones += total;
        __syncthreads();
    }
}

// one wave per member of list l of the old layout: to slot[r] of list l (side 0) or of list lnew (side 1)
// of the new layout, stored bytes, norm and id unchanged
__global__ __launch_bounds__(256) void split_scatter_kernel(const DevIndex *srcp, const DevIndex *dstp, uint32_t l,
                                                            uint32_t lnew, const int32_t *side, const uint32_t *slot,
                                                            uint32_t len)
{
    const DevIndex &src = *srcp, &dst = *dstp;
    const uint32_t r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= len) return;
    size_t ls, ld;
    const Arena &as = locate(src, l, r, ls);
    const Arena &ad = locate(dst, side[r] ? lnew : l, slot[r], ld);
    const int lane = threadIdx.x & 63, row_bytes = src.row_bytes;
    const uint4 *from = reinterpret_cast<const uint4 *>(as.vec + ls * (size_t)row_bytes);
    uint4 *to = reinterpret_cast<uint4 *>(ad.vec + ld * (size_t)row_bytes);
    for (int i = lane; i < row_bytes / 16; i += 64) to[i] = from[i];
    if (lane == 0) {
        ad.norm[ld] = as.norm[ls];
        ad.ids[ld] = as.ids[ls];
    }
}

hipError_t launch_split_list(const DevIndex *src, const DevIndex *dst, uint32_t l, uint32_t lnew, const int32_t *side,
                             uint32_t *slot, uint32_t len, hipStream_t s)
{
    if (len == 0) return hipSuccess;
    hipLaunchKernelGGL(split_slots_kernel, dim3(1), dim3(1024), 0, s, side, len, slot);
    hipLaunchKernelGGL(split_scatter_kernel, dim3((len + 3) / 4), dim3(256), 0, s, src, dst, l, lnew, side, slot, len);
    return hipGetLastError();
}

__global__ void copy_i32_kernel(const int32_t *src, int32_t *dst, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

hipError_t launch_copy_i32(const int32_t *src, int32_t *dst, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy_i32_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

} // namespace pk
