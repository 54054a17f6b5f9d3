// Lloyd's update step on the device, for index training (Section 2.2: the clusters of an IVF
// index come from k-means; Section 4.4 / 6.1 "IVF-Split" re-runs a light k-means on the GPU).
// The assignment step is the coarse search with nprobe = 1 under L2 (pk_api.hip); this file
// turns an assignment and its histogram into new centroids: exclusive scan, scatter of the row
// numbers into cluster-major order, then the members are summed in fp64, up to 256 of a cluster
// per workgroup (rows are read coalesced; the parts of a larger cluster meet by fp64 atomics), and every cluster divides its total.  An empty cluster keeps its
// centroid.  The objective of the assignment comes out of the same sums:
// sum_i |x_i - c|^2 = sum |x_i|^2 - 2 <c, sum x_i> + m |c|^2, in fp64.
#include <algorithm>
#include <type_traits>

#include "pk_internal.h"

namespace pk {

static_assert(PK_MAX_DIM <= 2 * 4 * 256, "a lane owns two times four dimensions at most");
constexpr int kKmChunk = 256;                     // members one workgroup sums
constexpr int kKmAhead = 8;                       // members in flight

__global__ __launch_bounds__(1024) void km_offsets_kernel(KmeansArgs a)
{
    __shared__ uint32_t s_wave[17];
    block_exscan(a.cnt, a.start, (uint32_t)a.nlist, s_wave);
    for (int l = threadIdx.x; l < a.nlist; l += 1024) a.piece0[l] = (a.cnt[l] + kKmChunk - 1) / kKmChunk;
    __syncthreads();
    const uint32_t pieces = block_exscan(a.piece0, a.piece0, (uint32_t)a.nlist, s_wave);
    if (threadIdx.x == 0) a.piece0[a.nlist] = pieces;
}

// Row numbers into cluster-major order.  A workgroup takes kKmRun rows, counts them per cluster in LDS and reserves
// each cluster's room with one atomic (an atomic per row on 162 words took 189 us for 262 144 rows).
constexpr int kKmRun = 2048;
__global__ __launch_bounds__(256) void km_scatter_kernel(KmeansArgs a, bool lds)
{
    extern __shared__ uint32_t s_at[];
    const int64_t i0 = (int64_t)blockIdx.x * kKmRun, i1 = i0 + kKmRun < a.n ? i0 + kKmRun : a.n;
    if (lds) {
        for (int l = threadIdx.x; l < a.nlist; l += 256) s_at[l] = 0u;
        __syncthreads();
        for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
            const uint32_t l = (uint32_t)a.assign[i];
            if (l < (uint32_t)a.nlist) atomicAdd(&s_at[l], 1u);
        }
        __syncthreads();
        for (int l = threadIdx.x; l < a.nlist; l += 256)
            if (s_at[l]) s_at[l] = a.start[l] + atomicAdd(&a.fill[l], s_at[l]);
        __syncthreads();
    }
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
        const uint32_t l = (uint32_t)a.assign[i];
        if (l >= (uint32_t)a.nlist) continue;
        const uint32_t at = lds ? atomicAdd(&s_at[l], 1u) : a.start[l] + atomicAdd(&a.fill[l], 1u);
        a.members[at] = (uint32_t)i;
    }
}

// One workgroup per piece: a cluster, or kKmChunk members of a longer one (a.piece0: pieces before each cluster).  A lane owns V
// neighbouring dimensions (T times, `across` lanes apart), `across` lanes a row, and the workgroup's 256 / across groups of
// lanes take every so manieth member; their sums meet in LDS.  The members' numbers are fetched once, so that the rows are the
// only memory operations of the loop, and a group's kKmAhead rows are requested before the first is added, by loads
// without a condition (with one, the compiler waits for each of them in turn).  Rows need no alignment: a lane's 16 bytes are the row's
// last ones where its dimensions reach past the end, and it keeps those that are its own.  A cluster of one piece is
// finished here, without atomics; the pieces of a longer one meet by float64 atomics, and km_finalize_kernel divides.
// With a lane per dimension and one group, 262 144 x 768, 4096 clusters took 247 us, now 180 (4.5 TB/s), 200 000 x 128, 1024 clusters 91
// and now 25, 100 000 x 1300, 300 clusters 188 and 141.
// ODD: some lane's dimensions reach past the row's end.
template <int V, int T, bool ODD>
__global__ __launch_bounds__(256) void km_accumulate_kernel(KmeansArgs a, uint32_t across)
{
    __shared__ double s_sum[256][V];
    __shared__ uint32_t s_member[kKmChunk];
    __shared__ double s_part[2][4];
    const uint32_t u = blockIdx.x, tid = threadIdx.x;
    if (u >= a.piece0[a.nlist]) return;
    uint32_t lo = 0, hi = (uint32_t)a.nlist - 1; // the last cluster whose pieces start at or before u
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (a.piece0[mid] <= u) lo = mid;
        else hi = mid - 1;
    }
    const uint32_t l = lo, cnt = a.cnt[l], first = (u - a.piece0[l]) * (uint32_t)kKmChunk;
    const uint32_t here = cnt - first < (uint32_t)kKmChunk ? cnt - first : (uint32_t)kKmChunk;
    s_member[tid] = a.members[a.start[l] + first + (tid < here ? tid : here - 1u)];
    static_assert(kKmChunk == 256, "a member per thread");
    __syncthreads();
    const uint32_t groups = 256u / across, group = tid / across, at = tid - group * across;
    int from[T]; // the lane's first dimension, and the first that it reads
    double sum[T][V] = {}, sq = 0.0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int j = (int)(at + across * t) * V;
        from[t] = j < a.d - V ? j : a.d - V;
    }
    auto own = [&](int t, int c) { return !ODD || from[t] + c >= (int)(at + across * t) * V; };
    // kKmAhead members from e0 on (FULL: there are that many; else the last one again where there is none, and not added)
    auto batch = [&](uint32_t e0, auto full) {
        constexpr bool FULL = decltype(full)::value;
        u32x4 v[kKmAhead][T];
#pragma unroll
        for (int w = 0; w < kKmAhead; ++w) {
            const uint32_t e = e0 + (uint32_t)w * groups;
            const float *const row = a.x + (size_t)s_member[FULL || e < here ? e : here - 1u] * a.d;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if constexpr (V == 4) v[w][t] = reinterpret_cast<const AnyFour *>(row + from[t])->v;
                else v[w][t][0] = __float_as_uint(row[from[t]]);
            }
        }
#pragma unroll
        for (int w = 0; w < kKmAhead; ++w) {
            const bool there = FULL || e0 + (uint32_t)w * groups < here; // (no branch: behind one, the load would be, too)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int c = 0; c < V; ++c) {
                    const double x = (double)__uint_as_float(there && own(t, c) ? v[w][t][c] : 0u);
                    sum[t][c] += x;
                    sq += x * x;
                }
        }
    };
    if (group < groups) {
        uint32_t e0 = group;
        for (; e0 + (uint32_t)(kKmAhead - 1) * groups < here; e0 += (uint32_t)kKmAhead * groups) batch(e0, std::true_type{});
        if (e0 < here) batch(e0, std::false_type{});
    }
    if constexpr (T == 1) { // (more than one group only then)
        if (groups > 1u) {
#pragma unroll
            for (int c = 0; c < V; ++c) s_sum[tid][c] = sum[0][c];
            __syncthreads();
            if (group == 0u)
                for (uint32_t g = 1; g < groups; ++g)
#pragma unroll
                    for (int c = 0; c < V; ++c) sum[0][c] += s_sum[g * across + at][c];
        }
    }
    const bool whole = cnt <= (uint32_t)kKmChunk;
    double obj = 0.0;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int w = 0; w < V; ++w) {
            const int j = from[t] + w;
            if (group != 0u || !own(t, w)) continue;
            if (whole) {
                float *c = a.centroids + (size_t)l * a.d + j;
                const double c0 = (double)*c;
                obj += (double)cnt * c0 * c0 - 2.0 * c0 * sum[t][w];
                *c = (float)(sum[t][w] / (double)cnt);
            } else {
                atomicAdd(&a.sums[(size_t)l * a.d + j], sum[t][w]);
            }
        }
    for (int off = 32; off > 0; off >>= 1) {
        sq += __shfl_xor(sq, off);
        obj += __shfl_xor(obj, off);
    }
    if ((tid & 63) == 0) {
        s_part[0][tid >> 6] = sq;
        s_part[1][tid >> 6] = obj;
    }
    __syncthreads();
    if (tid != 0) return;
    sq = (s_part[0][0] + s_part[0][1]) + (s_part[0][2] + s_part[0][3]);
    obj = (s_part[1][0] + s_part[1][1]) + (s_part[1][2] + s_part[1][3]);
    if (whole) atomicAdd(a.inertia, sq + obj);
    else atomicAdd(&a.sq[l], sq);
}

// clusters of several pieces: centroid = total / members, and the cluster's share of the objective of the assignment
// (a cluster of one piece is finished already; one without members keeps its centroid)
__global__ __launch_bounds__(256) void km_finalize_kernel(KmeansArgs a)
{
    __shared__ double s_part[4];
    const uint32_t l = blockIdx.x;
    const uint32_t m = a.cnt[l];
    if (m <= (uint32_t)kKmChunk) return;
    double obj = 0.0;
    for (int j = threadIdx.x; j < a.d; j += 256) {
        float *c = a.centroids + (size_t)l * a.d + j;
        const double c0 = (double)*c, sj = a.sums[(size_t)l * a.d + j];
        obj += (double)m * c0 * c0 - 2.0 * c0 * sj;
        *c = (float)(sj / (double)m);
    }
    for (int off = 32; off > 0; off >>= 1) obj += __shfl_xor(obj, off);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = obj;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(a.inertia, a.sq[l] + (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]));
}

hipError_t launch_kmeans_update(const KmeansArgs &a, hipStream_t s)
{
    if (a.n <= 0 || a.nlist <= 0 || a.d <= 0 || a.d > PK_MAX_DIM) return hipErrorInvalidValue;
    const bool lds = a.nlist <= kLdsLists;
    hipLaunchKernelGGL(km_offsets_kernel, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(km_scatter_kernel, dim3((uint32_t)((a.n + kKmRun - 1) / kKmRun)), dim3(256),
                       lds ? (size_t)a.nlist * 4 : 0, s, a, lds);
    const dim3 pieces((uint32_t)(a.n / kKmChunk + std::min<int64_t>(a.n, a.nlist) + 1)), threads(256); // at least as many as there are
    auto go = [&](auto kernel, int v) { // lanes per row: what it takes, or all of the workgroup's
        const uint32_t across = std::min(256u, (uint32_t)((a.d + v - 1) / v));
        hipLaunchKernelGGL(kernel, pieces, threads, 0, s, a, across);
    };
    if (a.d < 4) go(km_accumulate_kernel<1, 1, false>, 1);
    else if (a.d > 1024) go(km_accumulate_kernel<4, 2, true>, 4);
    else if (a.d % 4 == 0) go(km_accumulate_kernel<4, 1, false>, 4);
    else go(km_accumulate_kernel<4, 1, true>, 4);
    hipLaunchKernelGGL(km_finalize_kernel, dim3(a.nlist), dim3(256), 0, s, a);
    return hipGetLastError();
}

} // namespace pk
