// Coarse scoring for large query batches (and for build and k-means, where every vector is a
// "query"): S[m][n] = <Q_m, C_n> (inner product) or |C_n|^2 - 2 <Q_m, C_n> + |Q_m|^2
// (squared L2), Section 2.2's ranking of clusters by centroid distance, for all m, n.
//
// gemm_scores_kernel writes the scores: the coarse step of searches.  gemm_split_kernel finds every row's best
// column: the assignments of large inserts, of small sets and, of the rows that gemm_first_kernel leaves undecided, of other builds
// and k-means iterations.
//
// This is a dense contraction, so it runs on the matrix cores with fp32 inputs and fp32
// accumulation (v_mfma_f32_32x32x2_f32): no down-conversion of queries or centroids, so
// the probe ranking tracks the fp64 oracle to fp32 rounding.  128 x 128 output tile per
// workgroup (4 waves, 64 x 64 each as 2 x 2 MFMA blocks), K consumed 32 floats at a time
// through double-buffered LDS; both operands are row-major with the padded row stride of
// the scan layout, so K needs no tail handling.  As in the scan kernel the contraction
// index is permuted identically on both operands so that a lane's four consecutive floats
// (one ds_read_b128) feed four MFMAs.
#include <algorithm>
#include <type_traits>

#include "pk_internal.h"

namespace pk {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));

constexpr int kGemmTile = 128;
constexpr int kGemmBK = 32;               // floats per K step
constexpr int kGemmLdsStride = kGemmBK + 4; // floats; +4 keeps the b128 reads conflict free

// tiles of the kernel for few listed rows: 32 rows x 128 columns each
constexpr int kListRows = 32, kListCols = 128;
__device__ __forceinline__ uint32_t listed_tiles(uint32_t rows, int n_pad)
{
    return (rows + kListRows - 1) / kListRows * ((uint32_t)(n_pad + kListCols - 1) / kListCols);
}

// Four floats of a dense row of d from column `col` on: the load, and zeros past the row's end, which are put in when the floats
// are used, as putting them in waits for the load (see raw_load).
template <int RAW>
__device__ __forceinline__ f32x4 dense_load(const float *row, int col, int d)
{
    return __builtin_bit_cast(f32x4, raw_load<RAW>(reinterpret_cast<const uint32_t *>(row), col, d));
}
template <int RAW>
__device__ __forceinline__ f32x4 dense_zeros(f32x4 v, int col, int d)
{
    return __builtin_bit_cast(f32x4, raw_zeros<RAW>(__builtin_bit_cast(u32x4, v), col, d));
}

// f with the kind as a constant
template <typename F>
static auto for_raw(int kind, const F &f)
{
    switch (kind) {
    case kRawVec: return f(std::integral_constant<int, kRawVec>{});
    case kRawAny: return f(std::integral_constant<int, kRawAny>{});
    default: return f(std::integral_constant<int, kRawShort>{});
    }
}

// A wave's scores of listed rows into their best (value key, column): blocks of 32 columns x 32 rows, lane l holds, of row
// m0 + l % 32 of each block, columns n0 + (l / 32) * 4 + 8 * (r / 4) + r % 4.  One atomic per row: one per value, behind a
// look at the best so far, took 140 us of 311 rows and 4096 columns.
template <int MI, int NI>
__device__ __forceinline__ void best_of_listed(const GemmArgs &a, const f32x16 (&acc)[MI][NI], int m0, int n0, int rows, int lane)
{
    const int l32 = lane & 31, kg = lane >> 5;
    uint32_t row[MI], top[MI];
    int col[MI];
    float qn[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int m = m0 + i * 32 + l32;
        row[i] = a.list[m < rows ? m : rows - 1];
        top[i] = 0xffffffffu;
        col[i] = 0;
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) qn[i] = a.metric == PK_METRIC_L2 ? a.qnorm[row[i]] : 0.f;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        if (n0 + j * 32 >= a.n) continue; // (the same for the whole wave; the table has whole blocks of 32)
        f32x4 cn[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            cn[g] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (a.metric == PK_METRIC_L2) cn[g] = *reinterpret_cast<const f32x4 *>(a.cnorm + n0 + j * 32 + kg * 4 + g * 8);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int n = n0 + j * 32 + kg * 4 + 8 * (r >> 2) + (r & 3);
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                float v = acc[i][j][r];
                if (a.metric == PK_METRIC_L2) v = fmaxf(cn[r >> 2][r & 3] - 2.f * v + qn[i], 0.f);
                const uint32_t key = n < a.n ? min(order_bits(v, a.metric), kWorstKey) : 0xffffffffu;
                col[i] = key < top[i] ? n : col[i];
                top[i] = min(top[i], key);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        unsigned long long best = ((unsigned long long)top[i] << 32) | (uint32_t)col[i];
        const unsigned long long other = __shfl_xor(best, 32);
        best = other < best ? other : best;
        if (kg == 0 && m0 + i * 32 + l32 < rows && (uint32_t)(best >> 32) != 0xffffffffu) atomicMin(a.best + row[i], best);
    }
}

// LISTED: the rows are those of a list on the device (a.list, *a.nlisted of them, dense rows of a.d floats), and every row
// keeps its best (value key, column) by atomicMin instead of its scores; the grid walks the tiles there are.  For lists
// that fill tiles (see gemm_listed_kernel): 262 144 listed rows x 4096 x 768
// in 18.0 ms = 92 TFLOP/s, where the kernel for few of them took 82.
template <bool LISTED, int RAW = kRawVec>
__global__ __launch_bounds__(256) void gemm_scores_kernel(GemmArgs a)
{
    const int rows = LISTED ? (int)*a.nlisted : a.m;
    const uint32_t tn = (uint32_t)(a.n_pad + kGemmTile - 1) / kGemmTile;
    if constexpr (LISTED)
        if (listed_tiles((uint32_t)rows, a.n_pad) <= a.many) return;
    [[maybe_unused]] const uint32_t tiles = tn * ((uint32_t)(rows + kGemmTile - 1) / kGemmTile);
    __shared__ __align__(16) float sA[2][kGemmTile * kGemmLdsStride];
    __shared__ __align__(16) float sB[2][kGemmTile * kGemmLdsStride];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;        // wave's 64 x 64 quadrant
    const int l32 = lane & 31, kg = lane >> 5;      // MFMA row / column and k group
    const int ld = a.ld;                            // floats per row, multiple of 64
    const int ksteps = ld / kGemmBK;

    [[maybe_unused]] uint32_t t = blockIdx.x;
    do {
    const int m0 = (int)(LISTED ? t / tn : blockIdx.y) * kGemmTile, n0 = (int)(LISTED ? t % tn : blockIdx.x) * kGemmTile;
    // global -> register staging: each thread moves 4 x 16 B of A and of B per K step
    // row = (tid >> 3) + 32 * i, 16-byte column = tid & 7
    const int srow = tid >> 3, scol = (tid & 7) * 4;
    const float *ga[4], *gb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int ra = m0 + srow + 32 * i, rb = n0 + srow + 32 * i;
        ra = ra < rows ? ra : rows - 1; // clamp: rows past the end are computed and dropped
        rb = rb < a.n_pad ? rb : a.n_pad - 1;
        ga[i] = a.q + (LISTED ? (size_t)a.list[ra] * a.d : (size_t)ra * ld + scol);
        gb[i] = a.c + (size_t)rb * ld + scol;
    }
    f32x4 ra4[4], rb4[4];
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#define PK_GLOAD(ks)                                                                     \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                        \
    {                                                                                    \
        rb4[i] = *reinterpret_cast<const f32x4 *>(gb[i] + (size_t)(ks) * kGemmBK);       \
        if constexpr (LISTED) ra4[i] = dense_load<RAW>(ga[i], (ks) * kGemmBK + scol, a.d); \
        else ra4[i] = *reinterpret_cast<const f32x4 *>(ga[i] + (size_t)(ks) * kGemmBK);  \
    }
#define PK_LSTORE(buf, ks)                                                                               \
    _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                        \
    {                                                                                                    \
        if constexpr (LISTED) ra4[i] = dense_zeros<RAW>(ra4[i], (ks) * kGemmBK + scol, a.d);                  \
        *reinterpret_cast<f32x4 *>(&sA[buf][(srow + 32 * i) * kGemmLdsStride + scol]) = ra4[i];          \
        *reinterpret_cast<f32x4 *>(&sB[buf][(srow + 32 * i) * kGemmLdsStride + scol]) = rb4[i];          \
    }

    PK_GLOAD(0)
    PK_LSTORE(0, 0)
    __syncthreads();
    for (int ks = 0; ks < ksteps; ++ks) {
        const int buf = ks & 1;
        if (ks + 1 < ksteps) { PK_GLOAD(ks + 1) }
        const float *pa = &sA[buf][(wm * 64 + l32) * kGemmLdsStride + kg * 4];
        const float *pb = &sB[buf][(wn * 64 + l32) * kGemmLdsStride + kg * 4];
#pragma unroll
        for (int kc = 0; kc < kGemmBK / 8; ++kc) {
            f32x4 fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                fa[i] = *reinterpret_cast<const f32x4 *>(pa + i * 32 * kGemmLdsStride + kc * 8);
                fb[i] = *reinterpret_cast<const f32x4 *>(pb + i * 32 * kGemmLdsStride + kc * 8);
            }
#pragma unroll
            for (int j4 = 0; j4 < 4; ++j4)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) // (either way the same sums; a listed row's values belong into one lane)
                        acc[i][j] = LISTED ? __builtin_amdgcn_mfma_f32_32x32x2f32(fb[j][j4], fa[i][j4], acc[i][j], 0, 0, 0)
                                           : __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][j4], fb[j][j4], acc[i][j], 0, 0, 0);
        }
        if (ks + 1 < ksteps) {
            PK_LSTORE(buf ^ 1, ks + 1) // the other buffer was last read before the previous barrier
        }
        __syncthreads();
    }
#undef PK_GLOAD
#undef PK_LSTORE

    if constexpr (LISTED) {
        best_of_listed<2, 2>(a, acc, m0 + wm * 64, n0 + wn * 64, rows, lane);
        t += gridDim.x;
        continue;
    }
    // epilogue: lane holds column n = l32 of rows (kg*4 + 8*(r/4) + r%4) of each 32 x 32 block
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int n = n0 + wn * 64 + j * 32 + l32;
        if (n >= a.n_store) continue;
        const bool live = n < a.n;
        const float cn = (a.metric == PK_METRIC_L2 && live) ? a.cnorm[n] : 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + wm * 64 + i * 32 + kg * 4 + 8 * (r >> 2) + (r & 3);
                if (m < a.m) {
                    float v = acc[i][j][r];
                    if (a.metric == PK_METRIC_L2) v = fmaxf(cn - 2.f * v + a.qnorm[m], 0.f);
                    if (!live) v = a.metric == PK_METRIC_IP ? -INFINITY : INFINITY;
                    a.out[(size_t)m * a.stride + n] = v;
                }
            }
        }
    }
    } while (LISTED && t < tiles);
}

hipError_t launch_gemm_scores(const GemmArgs &a, hipStream_t s)
{
    if (a.m <= 0) return hipSuccess;
    if (a.ld % 64 != 0) return hipErrorInvalidValue;
    dim3 grid((a.n_pad + kGemmTile - 1) / kGemmTile, (a.m + kGemmTile - 1) / kGemmTile);
    hipLaunchKernelGGL(gemm_scores_kernel<false>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------- the same products on the 16-bit matrix cores

// An fp32 value as two halfs: x * 2^s = hi + lo + e with hi = half(x * 2^s), lo = half(x * 2^s - hi) and |e| at most
// 2^-23 of the value (2^-39 of the row's largest for values that are tiny beside it); s makes the row's largest value
// 2^14 .. 2^15, so nothing overflows.  A product is then hi hi + hi lo + lo hi (lo lo is below 2^-22 of it), three
// products of 11-bit numbers that are exact in fp32, at a sixteenth of the fp32 product's price each.
// Rows in memory: blocks of 32 elements, 64 bytes of hi then 64 bytes of lo; as many bytes as the fp32 row.

// Sum of a row in the order in which prep_row (pk_worklist.hip) adds its squares, whose thread i of 256 holds elements i, i + 256,
// ...  A wave's row: part[0][j] is the sum of the lane's elements 4 * lane + j, + 256, ....  A row of at most 256 elements on SUB lanes of a wave:
// part[u][j] is the lane's element 4 * lane + j + 4 * SUB * u.  (Elements there are none of add zeros, which change nothing.)  A
// query's norm is the same bits whichever kernel prepared it.
template <int SUB, int NP>
__device__ __forceinline__ float row_sum(float (&part)[NP][4])
{
    float sum = 0.f;
#pragma unroll
    for (int u = 0; u < NP; ++u) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) part[u][j] += __shfl_xor(part[u][j], off);
        const float w = (part[u][0] + part[u][2]) + (part[u][1] + part[u][3]);
#pragma unroll
        for (int at = 0; at < SUB; at += 16) {
            const float x = __shfl(w, at, SUB);
            sum = u == 0 && at == 0 ? x : sum + x;
        }
    }
    return sum;
}

// SUB lanes per row, of rows [0, m) from `x` (dense, d floats) or (CENT) of the n_c of the (padded) centroid table.  A lane has four
// elements of each of a row's T parts of 4 SUB.  top, top_left (of centroids): raised to the row's squared length and to what its first
// halfs leave out, as bits (not negative: in the order of the values).
// Bound by memory (300 000 rows of 4 KB read and written at 4.3 TB/s), and where rows are short by the rate at which workgroups
// start: with a wave per row, 32768 rows of up to 256 elements take 26 - 31 us, however short they are.  There several rows
// share a wave, and the workgroups stay and take row after row (long rows: 37 -> 40 us of 32768 x 768): 32768 x 128 27 -> 16 us.
template <int T, int SUB, bool CENT>
__device__ __forceinline__ void split_row(const SplitRowsArgs &a, const MultiArgs &mm, uint32_t r, int lane, uint32_t &top, uint32_t &top_left)
{
    static_assert(SUB == 64 || 4 * SUB * T <= 256, "rows that share a wave have 256 elements at most");
    constexpr int NP = SUB == 64 ? 1 : T; // sums that are kept apart (see row_sum)
    const int ld = a.ld, d = CENT ? ld : a.d;
    const float *src = CENT ? a.c + (size_t)r * ld : a.x + (size_t)r * d;
    const bool vec = (d & 3) == 0 && (reinterpret_cast<uintptr_t>(src) & 15) == 0; // (nearly always the same for the whole wave)
    f32x4 v[T];
    float big = 0.f, sq[NP][4] = {}, sq16[NP][4] = {}, off[NP][4] = {};
    if (vec) { // (all of a row's loads in flight at once: none of them under a condition)
#pragma unroll
        for (int t = 0; t < T; ++t) v[t] = dense_load<kRawVec>(src, lane * 4 + 4 * SUB * t, d);
#pragma unroll
        for (int t = 0; t < T; ++t) v[t] = dense_zeros<kRawVec>(v[t], lane * 4 + 4 * SUB * t, d);
    } else if (d >= 4) {
#pragma unroll
        for (int t = 0; t < T; ++t) v[t] = dense_load<kRawAny>(src, lane * 4 + 4 * SUB * t, d);
#pragma unroll
        for (int t = 0; t < T; ++t) v[t] = dense_zeros<kRawAny>(v[t], lane * 4 + 4 * SUB * t, d);
    } else {
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[t][j] = lane * 4 + 4 * SUB * t + j < d ? src[lane * 4 + 4 * SUB * t + j] : 0.f;
    }
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            big = fmaxf(big, fabsf(v[t][j]));
            sq[t % NP][j] += v[t][j] * v[t][j];
        }
    for (int o = SUB / 2; o > 0; o >>= 1) big = fmaxf(big, __shfl_xor(big, o));
    const float norm = row_sum<SUB>(sq);
    // 2^e <= big < 2^(e + 1); the scale stays a normal number (a row of zeros, or one below 2^-112, is scaled by 2^126)
    int s = 14 - ((int)(__float_as_uint(big) >> 23) - 127);
    s = s < -126 ? -126 : (s > 126 ? 126 : s);
    const float scale = __uint_as_float((uint32_t)(s + 127) << 23);
    char *dst = CENT ? a.cs : a.xs, *first = CENT ? a.ch : a.xh;
    if (dst) dst += (size_t)r * ld * 4; // (null: the rows are wanted in their other forms only)
    if (first) first += (size_t)r * ld * 2;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int i = lane * 4 + 4 * SUB * t;
        if (i >= ld) continue;
        half4 hi, lo;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float y = v[t][j] * scale; // exact
            hi[j] = (_Float16)y;
            const float rest = y - (float)hi[j]; // exact
            lo[j] = (_Float16)rest;
            off[t % NP][j] += rest * rest;
        }
        if (first) *reinterpret_cast<half4 *>(first + (size_t)i * 2) = hi;
        if (dst) {
            char *p = dst + (size_t)(i >> 5) * 128 + (i & 31) * 2;
            *reinterpret_cast<half4 *>(p) = hi;
            *reinterpret_cast<half4 *>(p + 64) = lo;
        }
        if (!CENT && a.copy) *reinterpret_cast<f32x4 *>(a.copy + (size_t)r * ld + i) = v[t];
    }
    if (!CENT && a.half_rows) { // the row as a half-precision index stores it: rounded to nearest even, norm of the rounded values
        char *h = a.half_rows + (size_t)r * a.half_bytes;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int i = lane * 4 + 4 * SUB * t;
            if (i * 2 >= a.half_bytes) continue;
            half4 w;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w[j] = (_Float16)v[t][j];
                const float f = (float)w[j];
                sq16[t % NP][j] += f * f;
            }
            *reinterpret_cast<half4 *>(h + (size_t)i * 2) = w;
        }
    }
    const float norm16 = row_sum<SUB>(sq16);
    const float rest = row_sum<SUB>(off);
    const float back = __uint_as_float((uint32_t)(127 - s) << 23);
    const float left = sqrtf(rest) * back; // length of what the first halfs leave out
    if constexpr (CENT) {
        if (lane == 0) a.c_back[r] = back;
        top = max(top, __float_as_uint(norm));
        top_left = max(top_left, __float_as_uint(left));
        return;
    }
    if (lane != 0) return;
    if (a.left) a.left[r] = left;
    if (a.x_back) a.x_back[r] = back;
    if (a.second) a.second[r] = 0xffffffffu;
    if (a.redo) a.redo[r] = ~0ull;
    if (a.qnorm) a.qnorm[r] = norm;
    if (a.half_rows) a.half_norm[r] = norm16;
    if (a.best) a.best[r] = ~0ull;
    if (a.meta.cand_off) {
        int h = 0;
        while (h + 1 < mm.n && r >= mm.qlo[h + 1]) ++h;
        a.meta.cand_off[r] = r * a.meta.stride;
        a.meta.cand_cnt[r] = (uint32_t)mm.ix[h]->nlist;
        a.meta.qagent[r] = (uint16_t)h;
    }
}

// The first workgroups take the centroids, and raise the largest lengths once each: the atomics meet at one word, 7 ns each, and
// hold up the other rows (one per centroid: the first 32768 rows x 768 with 4096 lists 66 us, with none 31; now 46).
template <int T, int SUB>
__global__ __launch_bounds__(256) void split_rows_kernel(SplitRowsArgs a, MultiArgs mm)
{
    const int lane = threadIdx.x & (SUB - 1);
    constexpr uint32_t kRows = 256 / SUB; // of a workgroup at a time
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < a.meta.nclear; i += gridDim.x * blockDim.x) a.meta.clear[i] = 0u;
    const uint32_t group = threadIdx.x / SUB, cents = (a.n_c + kRows - 1) / kRows;
    uint32_t top = 0, top_left = 0;
    if (blockIdx.x < cents) {
        __shared__ uint32_t s_top[2][4];
        const uint32_t r = blockIdx.x * kRows + group;
        if (r < a.n_c) split_row<T, SUB, true>(a, mm, r, lane, top, top_left);
        for (int off = SUB; off < 64; off <<= 1) {
            top = max(top, (uint32_t)__shfl_xor((int)top, off));
            top_left = max(top_left, (uint32_t)__shfl_xor((int)top_left, off));
        }
        if ((threadIdx.x & 63u) == 0) {
            s_top[0][threadIdx.x >> 6] = top;
            s_top[1][threadIdx.x >> 6] = top_left;
        }
        __syncthreads();
        uint32_t *const word = threadIdx.x == 0 ? a.cmax : threadIdx.x == 1 ? a.cmax_left : nullptr;
        if (!word) return;
        const uint32_t *const w = s_top[threadIdx.x];
        const uint32_t v = max(max(w[0], w[1]), max(w[2], w[3]));
        if (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < v) atomicMax(word, v);
        return;
    }
    uint32_t row = (blockIdx.x - cents) * kRows + group;
    if constexpr (SUB == 64) {
        if (row < a.m) split_row<T, SUB, false>(a, mm, row, lane, top, top_left);
    } else {
        for (; row < a.m; row += (gridDim.x - cents) * kRows) split_row<T, SUB, false>(a, mm, row, lane, top, top_left);
    }
}

constexpr uint32_t kSplitRowsGrid = 2048; // workgroups that stay: eight per CU
hipError_t launch_split_rows(const SplitRowsArgs &a, const MultiArgs &mm, hipStream_t s)
{
    if (a.m + a.n_c == 0) return hipSuccess;
    if (a.ld % 64 != 0 || a.ld > PK_MAX_DIM || a.d > a.ld) return hipErrorInvalidValue;
    if (a.half_rows && (a.half_bytes % 256 != 0 || a.half_bytes > PK_MAX_DIM * 2 || a.half_bytes < a.d * 2)) return hipErrorInvalidValue;
    using Kernel = void (*)(SplitRowsArgs, MultiArgs);
    static constexpr Kernel shorter[] = {split_rows_kernel<1, 16>, split_rows_kernel<1, 32>, split_rows_kernel<2, 32>, split_rows_kernel<2, 32>};
    static constexpr Kernel longer[] = {split_rows_kernel<2, 64>, split_rows_kernel<3, 64>, split_rows_kernel<4, 64>, split_rows_kernel<5, 64>,
                                        split_rows_kernel<6, 64>};
    static_assert(PK_MAX_DIM <= 6 * 256, "a row has six parts at most");
    const int wide = a.half_rows ? std::max(a.ld, a.half_bytes / 2) : a.ld; // (a half-precision row may be padded further)
    const uint32_t each = wide <= 64 ? 16u : wide <= 256 ? 8u : 4u; // rows of a workgroup at a time
    const uint32_t most = (a.m + each - 1u) / each, cents = (a.n_c + each - 1u) / each;
    if (wide <= 256) hipLaunchKernelGGL(shorter[(wide - 1) / 64], dim3(cents + std::min(most, kSplitRowsGrid)), dim3(256), 0, s, a, mm);
    else hipLaunchKernelGGL(longer[(wide + 255) / 256 - 2], dim3(cents + most), dim3(256), 0, s, a, mm);
    return hipGetLastError();
}

// What the value of a column that is no list begins with in the search for the best: larger than every list's (whose margins
// are infinite where it would not be).
constexpr float kNoList = 3.0e38f;

// One more value for the three smallest (low <= next <= third), and the place of the smallest.  As one statement, since the
// compiler would put the places off and keep every `low` until then; the two instructions between vcc's write and its read are those that
// the read has to wait.  (v_min_f32 because fminf would first quiet what might be a signalling NaN.)
__device__ __forceinline__ void lowest(float t, uint32_t here, float &low, float &next, float &third, uint32_t &at)
{
    asm("v_cmp_nlt_f32 vcc, %4, %0\n\t"
        "v_med3_f32 %2, %1, %2, %4\n\t"
        "v_med3_f32 %1, %0, %1, %4\n\t"
        "v_cndmask_b32 %3, %5, %3, vcc\n\t"
        "v_min_f32 %0, %0, %4"
        : "+&v"(low), "+&v"(next), "+&v"(third), "+&v"(at)
        : "v"(t), "i"(here)
        : "vcc");
}

// A wave's products (blocks of 32 columns x 32 rows: lane l holds, of row m0 + l % 32 of each block, columns
// n0 + (l / 32) * 4 + 8 * (r / 4) + r % 4) into the rows' best and near second values.  s_col: of the wave's columns.
template <int BN, int MI, int NI>
__device__ __forceinline__ void best_of_split(const SplitGemmArgs &a, const f32x16 (&acc)[MI][NI], const float *s_col, int m0, int n0, int rows,
                                              int lane, bool listed)
{
    const int l32 = lane & 31, kg = lane >> 5;
    if (n0 >= a.n) return; // no column of the wave's part is a list
    // t: smaller is nearer (inner product: -dot in the row's scale; L2: |c|^2 - 2 dot, the row's own norm left out)
    uint32_t row[MI];
    float factor[MI], low[MI], next[MI]; // (smallest t, smallest but one)
    int col[MI];                         // the smallest's first column inside the wave's part of the tile
    bool odd[MI];                        // a value that cannot be compared
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int m = m0 + i * 32 + l32 < rows ? m0 + i * 32 + l32 : rows - 1;
        row[i] = listed ? a.list[m] : (uint32_t)m;
        const float back = a.q_back[row[i]];
        factor[i] = a.metric == PK_METRIC_L2 ? -2.f * back : -1.f;
        low[i] = next[i] = INFINITY;
        col[i] = 0;
        odd[i] = false;
    }
    const float *const pc = s_col + kg * 4;
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 cb = *reinterpret_cast<const f32x4 *>(pc + j * 32 + g * 8);
            const f32x4 cn = *reinterpret_cast<const f32x4 *>(pc + BN + j * 32 + g * 8);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float t = fmaf(acc[i][j][g * 4 + e] * cb[e], factor[i], cn[e]);
                    odd[i] |= t != t;
                    col[i] = t < low[i] ? j * 32 + g * 8 + e : col[i];
                    next[i] = __builtin_amdgcn_fmed3f(low[i], next[i], t); // (low <= next)
                    low[i] = fminf(low[i], t);
                }
        }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        // the other half wave's columns of the row
        const float low2 = __shfl_xor(low[i], 32), next2 = __shfl_xor(next[i], 32);
        const int col1 = col[i] + kg * 4, col2 = __shfl_xor(col1, 32);
        odd[i] |= __shfl_xor((int)odd[i], 32) != 0;
        const bool mine = low[i] < low2 || (low[i] == low2 && col1 < col2);
        col[i] = mine ? col1 : col2;
        next[i] = fminf(fmaxf(low[i], low2), fminf(next[i], next2));
        low[i] = fminf(low[i], low2);
    }
    // either half wave goes on with every second block
    uint32_t met[MI], key[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int m = m0 + i * 32 + l32;
        met[i] = key[i] = 0xffffffffu;
        if (((i ^ kg) & 1) != 0 || m >= rows) continue;
        const float v = a.metric == PK_METRIC_IP ? -low[i] * a.q_back[row[i]] : low[i];
        key[i] = min(order_bits(v, a.metric), kWorstKey);
        const unsigned long long k = ((unsigned long long)key[i] << 32) | (uint32_t)(n0 + col[i]);
        met[i] = (uint32_t)(atomicMin(a.best + row[i], k) >> 32);
    }
    if (!a.second) return;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int m = m0 + i * 32 + l32;
        if (((i ^ kg) & 1) != 0 || m >= rows) continue;
        if (odd[i]) {
            atomicMin(a.second + row[i], kNoOrder);
            continue;
        }
        // the second best that this wave knows of: its own, or the worse of its best and the one it met (all ones: none)
        uint32_t other = max(met[i], key[i]);
        const float v = a.metric == PK_METRIC_IP ? -next[i] * a.q_back[row[i]] : next[i];
        other = min(other, min(order_bits(v, a.metric), kWorstKey));
        const float gap = fabsf(value_of(other, a.metric) - value_of(min(met[i], key[i]), a.metric));
        if (gap > near_margin(a.ld, a.metric, a.qnorm[row[i]], __uint_as_float(*a.cmax))) continue;
        atomicMin(a.second + row[i], gap == gap ? other : kNoOrder);
    }
}

// BM x BN output tile per workgroup of WM x WN waves; K in steps of 32 elements (128 bytes of a split row) through
// double-buffered LDS, fetched two steps ahead through two register stages (a step is short: 12 MFMAs of 32 cycles per
// 32 x 32 x 2 blocks, and the operands come from L2).  Every row keeps its best (value key, column) by atomicMin
// instead of writing scores: top-1 assignment, which then needs no score matrix (268 MB per 16384 rows x 4096) and no
// selection.  Where a second column is near a row's best (in one tile, or met in memory by the tile's atomic: of two tiles
// with near best values the later one sees the earlier) its value is kept too; the fp32 kernel then decides for the
// rows that end up with a near second, so that every assignment is the one that kernel makes.
// The centroids are the matrix instructions' first operand and the rows the second, so that a lane holds 16 columns of ONE
// row per block and looks for their best without a word to its neighbours: 6 instructions a value.  (With the rows first a
// row lay across 32 lanes, and the moves and ballots over them took 75 us of each launch: 658 -> 582 us.)
// All rows of large inserts and small sets, in tiles that give every CU one, and LISTED: rows that gemm_first_kernel leaves,
// listed fp32 rows that are split on their way into LDS; the grid walks the tiles there are.
// Bound by the chain of short steps: 256 x 256 tiles, eight waves on a CU, keep the matrix cores busy for half of the cycles
// and LDS for 20 % (no bank conflicts); waves wait for memory and barriers a third of their time.  32768 x 4096 x 768 in
// 582 us = 354 TFLOP/s of fp32 products (when every assignment took it; such sets begin with gemm_first_kernel now), where the
// fp32 kernel's chunk of 16384 took 962 us = 107 and its
// selection 194.  (Not for the coarse step of searches, 1024 x 4096 x 768 69 -> 39 us: a query's probes at a near tie would
// then depend on which kernel its call takes.)  By its own values alone,
// 28 rows came out on the wrong side of a near tie, against 64 bits, over seven sets of 0.5 - 1 M rows
// (64 <= d <= 1536), and 46 by the fp32 kernel's.
template <int BM, int BN, int WM, int WN, bool LISTED, int RAW>
__device__ __forceinline__ void split_tiles(const SplitGemmArgs &a, char *smem, int rows)
{
    constexpr int TH = WM * WN * 64;
    constexpr int MI = BM / WM / 32, NI = BN / WN / 32; // 32 x 32 blocks per wave
    constexpr int LD = 144;                             // LDS bytes per row: 128 + 16, conflict-free b128 reads
    constexpr int LOADS = (BM + BN) * 8 / TH;           // 16-byte pieces per thread and step
    static_assert((BM * 8) % TH == 0 && (BN * 8) % TH == 0, "a thread's piece is of A or of B for the whole workgroup");
    constexpr int ALOADS = BM * 8 / TH;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int l32 = lane & 31, kg = lane >> 5;
    const uint32_t tn = (uint32_t)(a.n_pad + BN - 1) / BN, tm = (uint32_t)(rows + BM - 1) / BM, total = tn * tm;
    float *const s_col = reinterpret_cast<float *>(smem + (size_t)2 * (BM + BN) * LD); // [2][BN]
    char *const put = smem + (size_t)(tid >> 3) * LD + (tid & 7) * 16;
    constexpr int ROWS_PER = TH / 8; // LDS rows between a thread's pieces
    const int steps = a.ld / 32;
    const size_t row_bytes = (size_t)a.ld * 4;

    for (uint32_t b = blockIdx.x; b < total; b += gridDim.x) {
    // XCD-aware order: workgroups go to the 8 XCDs in turn; each XCD takes one contiguous part of the tiles, and walks
    // it in groups of 8 tile rows, so that the tiles in flight on an XCD share their rows and columns in its L2
    const uint32_t xcd = b & 7u, per = total / 8u, extra = total % 8u;
    const uint32_t t = xcd * per + (xcd < extra ? xcd : extra) + (b >> 3);
    constexpr uint32_t GM = 8;
    const uint32_t grp = t / (GM * tn), in = t - grp * GM * tn;
    const uint32_t gm = tm - grp * GM < GM ? tm - grp * GM : GM;
    const int m0 = (int)(grp * GM + in % gm) * BM, n0 = (int)(in / gm) * BN;

    const char *src[LOADS];
    [[maybe_unused]] float scale[ALOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int piece = i < ALOADS ? tid + i * TH : tid + (i - ALOADS) * TH;
        int r = (i < ALOADS ? m0 : n0) + (piece >> 3);
        const int last = i < ALOADS ? rows - 1 : a.n_pad - 1;
        r = r < last ? r : last; // rows past the end are computed and dropped
        if (LISTED && i < ALOADS) {
            const uint32_t row = a.list[r];
            src[i] = reinterpret_cast<const char *>(a.x + (size_t)row * a.d);
            scale[i] = 1.f / a.q_back[row]; // (a power of two: exact)
        } else {
            src[i] = (i < ALOADS ? a.q : a.c) + (size_t)r * row_bytes + (piece & 7) * 16;
        }
    }
    u32x4 s0[LOADS], s1[LOADS];
    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // (past the last step the last one is fetched again: every load is unconditional)
    auto fetch = [&](u32x4 (&st)[LOADS], int ks) {
        ks = ks < steps ? ks : steps - 1;
        const size_t at = (size_t)ks * 128;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            if (LISTED && i < ALOADS)
                st[i] = __builtin_bit_cast(u32x4, dense_load<RAW>(reinterpret_cast<const float *>(src[i]), ks * 32 + (tid & 7) * 4, a.d));
            else
                st[i] = *reinterpret_cast<gvec4>(in_global(src[i]) + at);
        }
    };
    auto store = [&](const u32x4 (&st)[LOADS], int buf, [[maybe_unused]] int ks) {
        char *const to = put + (size_t)buf * (BM + BN) * LD;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            if (LISTED && i < ALOADS) { // 4 floats: their first halfs into the row's first 64 bytes, the rest behind
                const f32x4 v = dense_zeros<RAW>(__builtin_bit_cast(f32x4, st[i]), ks * 32 + (tid & 7) * 4, a.d);
                half4 hi, lo;
#pragma unroll
                for (int j = 0; j < 4; ++j) { // (the same values as split_rows_kernel's)
                    const float y = v[j] * scale[i];
                    hi[j] = (_Float16)y;
                    lo[j] = (_Float16)(y - (float)hi[j]);
                }
                char *const p = to + (size_t)i * ROWS_PER * LD - (tid & 7) * 8;
                *reinterpret_cast<half4 *>(p) = hi;
                *reinterpret_cast<half4 *>(p + 64) = lo;
            } else {
                *reinterpret_cast<u32x4 *>(to + (size_t)i * ROWS_PER * LD) = st[i];
            }
        }
    };
    auto step = [&](int buf) {
        const char *pa = smem + (size_t)buf * (BM + BN) * LD + (size_t)(wm * (BM / WM) + l32) * LD + kg * 16;
        const char *pb = smem + (size_t)buf * (BM + BN) * LD + (size_t)(BM + wn * (BN / WN) + l32) * LD + kg * 16;
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
            half8 ah[MI], al[MI], bh[NI], bl[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                ah[i] = *reinterpret_cast<const half8 *>(pa + i * 32 * LD + kc * 32);
                al[i] = *reinterpret_cast<const half8 *>(pa + i * 32 * LD + kc * 32 + 64);
            }
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                bh[j] = *reinterpret_cast<const half8 *>(pb + j * 32 * LD + kc * 32);
                bl[j] = *reinterpret_cast<const half8 *>(pb + j * 32 * LD + kc * 32 + 64);
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh[j], al[i], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bl[j], ah[i], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh[j], ah[i], acc[i][j], 0, 0, 0);
        }
    };
    fetch(s0, 0);
    fetch(s1, 1);
    if constexpr (LISTED) __syncthreads(); // the tile before is done with LDS
    store(s0, 0, 0);
    fetch(s0, 2);
    // per column: what undoes its scale, and what its product is added to (a column that is no list comes behind every list)
    if (tid < BN) {
        const int n = n0 + tid;
        s_col[tid] = n < a.n ? a.c_back[n] : 0.f;
        s_col[BN + tid] = n < a.n ? (a.metric == PK_METRIC_L2 ? a.cnorm[n] : 0.f) : INFINITY;
    }
    __syncthreads();
    for (int ks = 0; ks < steps; ks += 2) { // steps is even: rows are padded to 64 elements
        step(0);
        store(s1, 1, ks + 1); // (buffer 1 was last read before the barrier that ended the step before)
        fetch(s1, ks + 3);
        __syncthreads();
        step(1);
        store(s0, 0, ks + 2);
        fetch(s0, ks + 4);
        __syncthreads();
    }
    best_of_split<BN, MI, NI>(a, acc, s_col + wn * (BN / WN), m0 + wm * (BM / WM), n0 + wn * (BN / WN), rows, lane, LISTED);
    if constexpr (!LISTED) return;
    }
}

template <int BM, int BN, int WM, int WN, bool LISTED, int RAW = kRawVec>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(2))) void gemm_split_kernel(SplitGemmArgs a)
{
    extern __shared__ __align__(16) char smem[]; // [2][BM + BN][144], then [2][BN] floats
    if (a.skipped && *a.skipped > a.skip_from) return; // near ties are the rule: the next kernel takes these rows whole
    const int rows = LISTED ? (int)*a.nlisted : a.m;
    if constexpr (LISTED) {
        // Few rows are bound by the steps of one tile (64 x 64: 0.6 us per 32 elements, 128 x 128: 1.0): quarter tiles while the
        // grid takes them all at once.  300 000 x 1024, what is left of a chunk for 512 lists 32 -> 21 us, 262 144 x 768 for 4096
        // 29 -> 17; two rounds of them take as long as one of the others.
        const uint32_t quarters = (uint32_t)((a.n_pad + 63) / 64) * (uint32_t)((rows + 63) / 64);
        if (quarters <= gridDim.x) {
            split_tiles<64, 64, 2, 2, true, RAW>(a, smem, rows);
            return;
        }
    }
    split_tiles<BM, BN, WM, WN, LISTED, RAW>(a, smem, rows);
}

// A wave's products of first halfs into the rows' best, second best and third: as best_of_split, but the three smallest values and
// the column of the smallest cost seven instructions a value.  The second's column is looked for, by its value, only where the second
// is near the row's best so far.  (Six with the column in the value's last five bits, which is then no longer the 32-bit sum that
// it was: gemm_first_kernel 244 us instead of 250.)  s_col, s_row: of the wave's columns and rows.
template <int BM, int BN, int MI, int NI>
__device__ __forceinline__ void best_of_first(const SplitGemmArgs &a, f32x16 (&acc)[MI][NI], const float *s_col, const float *s_row, int m0,
                                              int n0, int lane)
{
    const int l32 = lane & 31, kg = lane >> 5;
    if (n0 >= a.n) return; // no column of the wave's part is a list
    // t: smaller is nearer (inner product: -dot in the row's scale; L2: |c|^2 - 2 dot, the row's own norm left out)
    float factor[MI], low[MI], next[MI], third[MI];
    uint32_t at[MI]; // the smallest one's place among the lane's columns
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        factor[i] = a.metric == PK_METRIC_L2 ? -2.f * s_row[i * 32 + l32] : -1.f;
        low[i] = next[i] = third[i] = kNoList;
        at[i] = 0;
    }
    const float *const pc = s_col + kg * 4;
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 cb = *reinterpret_cast<const f32x4 *>(pc + j * 32 + g * 8);
            const f32x4 cn = *reinterpret_cast<const f32x4 *>(pc + BN + j * 32 + g * 8);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const float t = fmaf(acc[i][j][g * 4 + e] * cb[e], factor[i], cn[e]);
                    lowest(t, j * 16 + g * 4 + e, low[i], next[i], third[i], at[i]);
                    acc[i][j][g * 4 + e] = t;
                }
        }
    auto column = [&](uint32_t place, int half) { // of the tile
        return (uint32_t)n0 + (place >> 4) * 32u + ((place >> 2) & 3u) * 8u + (place & 3u) + (uint32_t)half * 4u;
    };
    auto key_of = [&](float t, float back) { return min(order_bits(a.metric == PK_METRIC_IP ? -t * back : t, a.metric), kWorstKey); };
    // either half wave goes on with every second block: the other's columns of its rows, and the row's best so far
    constexpr uint32_t kLater = 0xffffffffu; // col2: the second best is not the smallest of either half, and where it is not known yet
    unsigned long long mine[MI], met[MI];
    float t2[MI], t3[MI];
    uint32_t col2[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const float low2 = __shfl_xor(low[i], 32), next2 = __shfl_xor(next[i], 32), third2 = __shfl_xor(third[i], 32);
        const uint32_t at2 = (uint32_t)__shfl_xor((int)at[i], 32);
        const bool first = low[i] <= low2;
        const float t1 = first ? low[i] : low2, u = first ? low2 : low[i], w = fminf(next[i], next2);
        t2[i] = u <= w ? u : w;
        t3[i] = fminf(fminf(third[i], third2), fminf(fmaxf(low[i], next2), fmaxf(next[i], low2)));
        mine[i] = ((unsigned long long)key_of(t1, s_row[i * 32 + l32]) << 32) | column(first ? at[i] : at2, first ? kg : kg ^ 1);
        col2[i] = u <= w ? column(first ? at2 : at[i], first ? kg ^ 1 : kg) : kLater;
        met[i] = ~0ull;
        if (((i ^ kg) & 1) == 0 && m0 + i * 32 + l32 < a.m) met[i] = atomicMin(a.best + m0 + i * 32 + l32, mine[i]);
    }
    // Whoever comes behind goes on to the next word (every value but a word's last least leaves it once), unless it is too
    // far from the best so far to matter.  With three near ones in the wave alone the row has more than two candidates, and the
    // better of those behind the best says so (it stays near a better best as long as any of them does).
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int m = m0 + i * 32 + l32;
        const bool own = ((i ^ kg) & 1) == 0 && m < a.m;
        const float margin = s_row[BM + i * 32 + l32], back = s_row[i * 32 + l32];
        const unsigned long long lead = mine[i] < met[i] ? mine[i] : met[i], behind = mine[i] < met[i] ? met[i] : mine[i];
        const float best = value_of((uint32_t)(lead >> 32), a.metric);
        auto near = [&](uint32_t key) { return key != 0xffffffffu && !(fabsf(value_of(key, a.metric) - best) > margin); };
        auto enter = [&](unsigned long long k) {
            const unsigned long long old = atomicMin(a.next + m, k);
            const uint32_t out = (uint32_t)((old < k ? k : old) >> 32);
            if (out != 0xffffffffu) atomicMin(a.second + m, out);
        };
        const uint32_t key1 = (uint32_t)(behind >> 32), key2 = key_of(t2[i], back);
        const bool many = own && near(key_of(t3[i], back)), two = own && !many && near(key2);
        if (__any(two && col2[i] == kLater)) {
            // The second one's place, by its value.  It is in the half of the best, whose place is the first of those with the
            // smallest value: of several that are as large the last is another one.
            uint32_t place = kLater;
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) place = acc[i][j][e] == t2[i] ? (uint32_t)(j * 16 + e) : place;
            const uint32_t place2 = (uint32_t)__shfl_xor((int)place, 32);
            if (col2[i] == kLater) col2[i] = place != kLater ? column(place, kg) : column(place2, kg ^ 1);
        }
        if (many) atomicMin(a.second + m, min(key1, key2));
        if (!own || many) continue;
        if (near(key1)) enter(behind);
        if (two) enter(((unsigned long long)key2 << 32) | col2[i]);
    }
}

// The products of the first halfs alone: what decides all but a few rows of an assignment, at a third of the price.
// Same tiles and order as gemm_split_kernel; the operands go from memory into LDS without registers in between
// (one instruction per wave moves 16 rows x 64 bytes), three steps of 32 elements ahead of the one being multiplied, in
// four buffers.  The 16-byte pieces of a row lie in the order piece ^ ((row >> 1) & 3), so that the reads of a piece of 8
// consecutive rows meet no bank twice.  The loads are counted by hand (the compiler would wait for all of them before the
// next LDS read): they are the only memory operations of a tile's steps, complete in order, and a
// step's have arrived when at most those of the two steps behind it are outstanding (operations between two tiles only make
// the count stricter).  Workgroups stay and walk the tiles: the last steps of a tile request the first ones of the next, and
// its rows' and columns' factors are fetched before the search for the best, so that only that search (a fifth of the time)
// leaves the matrix cores idle.
// Rows keep their best two columns, and whether a third is near: two candidates are settled by pair_ties_kernel, more by the
// products of the whole values.
// 32768 x 4096 x 768 in 247 - 252 us = 825 TFLOP/s (six instructions a value in the search, with less than the whole value, 242 - 246 on the
// same boxes; a workgroup per tile and eight instructions 252 where the six took 235);
// a large library product of halfs runs at 1390 here.  150 us go to the matrix instructions at the clock they leave (timed
// alone), and what else is done adds to that as if one after the other: with the two waves of a SIMD taking turns to read and to
// multiply, a barrier between, and pieces in an order without bank conflicts, 234; two workgroups per CU with tiles of half the size
// (249 of 252), three buffers (247) and operands read ahead (253) change nothing, waves of 128 x 128, one per SIMD, take 289.
// A k-means iteration of 262 144 rows over 4096 lists 3560 -> 3000 us (a tenth of its rows have two candidates, for which
// the products of the whole values took 0.49 ms, pair_ties_kernel takes 0.06), with every list given twice 15.9 -> 4.7 ms.
template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(2))) void gemm_first_kernel(SplitGemmArgs a)
{
    constexpr int TH = WM * WN * 64;
    constexpr int MI = BM / WM / 32, NI = BN / WN / 32;
    constexpr int STEP = (BM + BN) * 64;            // bytes of one step's buffer
    constexpr int LOADS = STEP / 16 / TH;           // loads per wave and step
    constexpr int ALOADS = BM * 64 / 16 / TH;       // ... of them of rows (the others: of centroids)
    static_assert((BM * 4) % TH == 0 && (BN * 4) % TH == 0, "a load is of A or of B for the whole workgroup");
    static_assert(TH >= BM + BN, "a thread per column and row of a tile");
    extern __shared__ __align__(16) char smem[]; // [4][BM + BN][64], then [2][2][BN + BM] floats
    if (a.skipped && *a.skipped > a.skip_from) return; // near ties are the rule: the next kernel takes these rows whole
    if (a.skipped2 && *a.skipped2 > a.skip_from2) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int l32 = lane & 31, kg = lane >> 5;
    const uint32_t tn = (uint32_t)(a.n_pad + BN - 1) / BN, tm = (uint32_t)(a.m + BM - 1) / BM, total = tn * tm;
    auto place = [&](uint32_t b, int &m0, int &n0) { // (the order of gemm_split_kernel; b % 8 stays a workgroup's XCD)
        const uint32_t xcd = b & 7u, per = total / 8u, extra = total % 8u;
        const uint32_t t = xcd * per + (xcd < extra ? xcd : extra) + (b >> 3);
        constexpr uint32_t GM = 8;
        const uint32_t grp = t / (GM * tn), in = t - grp * GM * tn;
        const uint32_t gm = tm - grp * GM < GM ? tm - grp * GM : GM;
        m0 = (int)(grp * GM + in % gm) * BM;
        n0 = (int)(in / gm) * BN;
    };

    const int steps = a.ld / 32; // (two at least: rows are padded to 64 elements)
    const uint32_t row_bytes = (uint32_t)a.ld * 2u;
    // what is requested next: step rk of tile rb, into buffer rg % 4
    uint32_t rb = blockIdx.x, rg = 0, off[LOADS];
    int rk = 0;
    const char *base_a, *base_b;
    auto aim = [&]() {
        int m0, n0;
        place(rb, m0, n0);
        base_a = a.q + (size_t)m0 * row_bytes;
        base_b = a.c + (size_t)n0 * row_bytes;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int piece = (i < ALOADS ? i : i - ALOADS) * TH + tid; // of the operand's part of the buffer: row piece / 4
            int r = piece >> 2;
            const int p = (piece & 3) ^ ((r >> 1) & 3);
            const int last = i < ALOADS ? a.m - 1 - m0 : a.n_pad - 1 - n0;
            r = r < last ? r : last; // rows past the end are computed and dropped
            off[i] = (uint32_t)r * row_bytes + (uint32_t)p * 16u;
        }
    };
    // where this wave's loads of a step go: 1024 bytes each, lane by lane
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem + (uint32_t)wave * 1024u;
    auto request = [&]() {
        const char *const pa = base_a + rk * 64, *const pb = base_b + rk * 64;
        const uint32_t to = lds0 + (rg & 3u) * STEP;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) // (m0 is where the loads go, and an operand, so that the compiler knows what it holds)
            asm volatile("s_nop 0\n\t"
                         "global_load_lds_dwordx4 %1, %2"
                         :
                         : "{m0}"(to + (uint32_t)i * (TH * 16)), "v"(off[i]), "s"(i < ALOADS ? pa : pb)
                         : "memory");
        ++rg;
        if (rk + 1 < steps) {
            ++rk;
        } else if (rb + gridDim.x < total) {
            rk = 0;
            rb += gridDim.x;
            aim();
        } // (past the last tile's last step that step again: the count of loads is the same for every step)
    };
    // Per column: what undoes its scale, and what its product is added to (a column that is no list comes behind every list);
    // per row: what undoes its scale, and what values may differ by and still change places.  Fetched a tile ahead.
    const float cmax = __uint_as_float(*a.cmax), cmax_left = __uint_as_float(*a.cmax_left);
    float f0 = 0.f, f1 = 0.f, f2 = 0.f;
    auto fetch_factors = [&](uint32_t b) {
        int m0, n0;
        place(b, m0, n0);
        if (tid < BN) {
            const int n = n0 + tid;
            const int c = n < a.n ? n : 0;
            f0 = a.c_back[c];
            f1 = a.metric == PK_METRIC_L2 ? a.cnorm[c] : 0.f;
            f2 = n < a.n ? 1.f : 0.f;
        } else if (tid < BN + BM) {
            const int m = m0 + tid - BN;
            const int r = m < a.m ? m : a.m - 1;
            f0 = a.q_back[r];
            f1 = a.qnorm[r];
            f2 = a.left[r];
        }
    };
    float *const s_factors = reinterpret_cast<float *>(smem + 4 * STEP);
    auto put_factors = [&](int parity) {
        float *const to = s_factors + parity * 2 * (BN + BM);
        if (tid < BN) {
            to[tid] = f2 != 0.f ? f0 : 0.f;
            to[BN + tid] = f2 != 0.f ? f1 : kNoList;
        } else if (tid < BN + BM) {
            to[2 * BN + tid - BN] = f0;
            to[2 * BN + BM + tid - BN] = first_margin(a.ld, a.metric, f1, cmax, f2, cmax_left);
        }
    };
    // byte offsets inside a buffer of the 16 bytes that the lane reads of a block's row, in each half of a step
    const uint32_t sw = (uint32_t)((l32 >> 1) & 3);
    const uint32_t at0 = (uint32_t)l32 * 64u + (((uint32_t)kg) ^ sw) * 16u, at1 = (uint32_t)l32 * 64u + (((uint32_t)kg + 2u) ^ sw) * 16u;
    fetch_factors(rb); // (the grid has no more workgroups than there are tiles)
    aim();
    request();
    request();
    request();
    uint32_t gs = 0; // steps done
    int parity = 0;
    for (uint32_t b = blockIdx.x; b < total; b += gridDim.x, parity ^= 1) {
        put_factors(parity); // (read after this tile's barriers; the other half may still be read by waves a tile behind)
        f32x16 acc[MI][NI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        for (int ks = 0; ks < steps; ++ks, ++gs) {
            // this step's operands are there (this wave's by its count, the others' by the barrier), and every wave has read
            // what it wanted of the step before, whose buffer the next request fills
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(2 * LOADS) : "memory");
            request();
            const char *const buf = smem + (gs & 3u) * STEP;
            const char *const pa = buf + wm * (BM / WM) * 64, *const pb = buf + (BM + wn * (BN / WN)) * 64;
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) {
                const uint32_t at = kc ? at1 : at0;
                half8 ah[MI], bh[NI];
#pragma unroll
                for (int i = 0; i < MI; ++i) ah[i] = *reinterpret_cast<const half8 *>(pa + at + i * 32 * 64);
#pragma unroll
                for (int j = 0; j < NI; ++j) bh[j] = *reinterpret_cast<const half8 *>(pb + at + j * 32 * 64);
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh[j], ah[i], acc[i][j], 0, 0, 0);
            }
        }
        if (b + gridDim.x < total) fetch_factors(b + gridDim.x);
        int m0, n0;
        place(b, m0, n0);
        const float *const s_col = s_factors + parity * 2 * (BN + BM);
        best_of_first<BM, BN, MI, NI>(a, acc, s_col + wn * (BN / WN), s_col + 2 * BN + wm * (BM / WM), m0 + wm * (BM / WM), n0 + wn * (BN / WN), lane);
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory"); // nothing may still be on its way into LDS when the workgroup ends
}

template <int BM, int BN, int WM, int WN>
static hipError_t launch_split_one(const SplitGemmArgs &a, [[maybe_unused]] int num_cu, hipStream_t s)
{
    static LdsCleared cleared, cleared_first;
    const int tiles = (a.n_pad + BN - 1) / BN * ((a.m + BM - 1) / BM);
    if (a.left) { // as many workgroups as the CUs hold at a time, whole rounds of the XCDs
        const int hold = std::max(num_cu / 8 * 8, 8) * (BM == 256 ? 1 : BM == 128 ? 2 : 4);
        return launch_with_lds(&gemm_first_kernel<BM, BN, WM, WN>, cleared_first, 4 * (BM + BN) * 64 + 4 * (BN + BM) * 4, a, std::min(tiles, hold),
                               WM * WN * 64, s);
    }
    return launch_with_lds(&gemm_split_kernel<BM, BN, WM, WN, false>, cleared, 2 * (BM + BN) * 144 + 2 * BN * 4, a, tiles, WM * WN * 64, s);
}

static bool split_gemm_valid(const SplitGemmArgs &a)
{
    return a.ld % 64 == 0 && a.n >= 1 && a.n <= a.n_pad && a.best && !(a.second && !(a.cmax && a.qnorm)) && !a.left == !a.cmax_left && !a.left == !a.next;
}

hipError_t launch_gemm_split(const SplitGemmArgs &a, int num_cu, hipStream_t s)
{
    if (a.m <= 0) return hipSuccess;
    if (!split_gemm_valid(a)) return hipErrorInvalidValue;
    auto tiles = [&](int b) { return (int64_t)((a.m + b - 1) / b) * ((a.n_pad + b - 1) / b); };
    // the largest tile that still gives every CU one
    if (tiles(256) >= num_cu) return launch_split_one<256, 256, 2, 4>(a, num_cu, s);
    if (tiles(128) >= num_cu) return launch_split_one<128, 128, 2, 2>(a, num_cu, s);
    return launch_split_one<64, 64, 2, 2>(a, num_cu, s);
}

hipError_t launch_gemm_split_listed(const SplitGemmArgs &a, int num_cu, hipStream_t s)
{
    if (!split_gemm_valid(a) || a.left || !a.list || !a.nlisted || !a.x || a.d > a.ld || a.d < 1) return hipErrorInvalidValue;
    constexpr int lds = 2 * 256 * 144 + 2 * 128 * 4;
    return for_raw(raw_kind(a.x, a.d), [&](auto raw) {
        static LdsCleared cleared;
        return launch_with_lds(&gemm_split_kernel<128, 128, 2, 2, true, raw()>, cleared, lds, a, 2 * num_cu, 256, s);
    });
}

// The fp32 products of a few listed rows (a.list, *a.nlisted of them: dense rows of a.d floats) with every column, in
// gemm_scores_kernel's order of operations, so that the values are the same; every row keeps its best (value key,
// column) by atomicMin.  Usually some hundred rows: bound by the latency of one tile, so a tile is 32 x 128 (a wave
// 32 x 32: 16 MFMAs per step of 32 elements), its operands are requested two steps ahead, and the grid walks the tiles
// there are.  As a form of the 128 x 128 kernel it took 210 us for whatever few rows there were; now 41 us for 311 rows of
// 768 against 4096 columns (140 with zeros put in as the rows were loaded, which waited for each load, and an atomic per value).  Lists of more than a.many tiles (two
// rounds of the grid, then longer than one round of 128 x 128 tiles) are gemm_scores_kernel<true>'s, and one of the two
// launches ends at once.
template <int RAW>
__global__ __launch_bounds__(256) void gemm_listed_kernel(GemmArgs a)
{
    __shared__ __align__(16) float sA[2][kListRows * kGemmLdsStride];
    __shared__ __align__(16) float sB[2][kListCols * kGemmLdsStride];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, kg = lane >> 5;
    const int ld = a.ld, ksteps = ld / kGemmBK; // even: rows are padded to 64 floats
    const int rows = (int)*a.nlisted;
    if (listed_tiles((uint32_t)rows, a.n_pad) > a.many) return;
    const uint32_t tn = (uint32_t)(a.n_pad + kListCols - 1) / kListCols, tm = (uint32_t)(rows + kListRows - 1) / kListRows;
    const int srow = tid >> 3, scol = (tid & 7) * 4;
    for (uint32_t t = blockIdx.x; t < tm * tn; t += gridDim.x) {
        const int m0 = (int)(t / tn) * kListRows, n0 = (int)(t % tn) * kListCols;
        const int mr = m0 + srow < rows ? m0 + srow : rows - 1; // clamp: rows past the end are computed and dropped
        const float *ga = a.q + (size_t)a.list[mr] * a.d, *gb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int rb = n0 + srow + 32 * i;
            rb = rb < a.n_pad ? rb : a.n_pad - 1;
            gb[i] = a.c + (size_t)rb * ld + scol;
        }
        f32x4 a0, a1, b0[4], b1[4];
        f32x16 acc[1][1];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
        auto fetch = [&](f32x4 &ra, f32x4 (&rb)[4], int ks) {
            const int at = (ks < ksteps ? ks : ksteps - 1) * kGemmBK; // (past the last step the last one again)
#pragma unroll
            for (int i = 0; i < 4; ++i) rb[i] = *reinterpret_cast<const f32x4 *>(gb[i] + at);
            ra = dense_load<RAW>(ga, at + scol, a.d); // the caller's rows: no padding, any alignment
        };
        auto put = [&](const f32x4 &ra, const f32x4 (&rb)[4], int buf, int ks) {
            *reinterpret_cast<f32x4 *>(&sA[buf][srow * kGemmLdsStride + scol]) = dense_zeros<RAW>(ra, ks * kGemmBK + scol, a.d);
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4 *>(&sB[buf][(srow + 32 * i) * kGemmLdsStride + scol]) = rb[i];
        };
        auto step = [&](int buf) {
            const float *pa = &sA[buf][l32 * kGemmLdsStride + kg * 4];
            const float *pb = &sB[buf][(wave * 32 + l32) * kGemmLdsStride + kg * 4];
#pragma unroll
            for (int kc = 0; kc < kGemmBK / 8; ++kc) {
                const f32x4 fa = *reinterpret_cast<const f32x4 *>(pa + kc * 8), fb = *reinterpret_cast<const f32x4 *>(pb + kc * 8);
#pragma unroll
                for (int j4 = 0; j4 < 4; ++j4) acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[j4], fa[j4], acc[0][0], 0, 0, 0);
            }
        };
        __syncthreads(); // the tile before is done with LDS
        fetch(a0, b0, 0);
        fetch(a1, b1, 1);
        put(a0, b0, 0, 0);
        fetch(a0, b0, 2);
        __syncthreads();
        for (int ks = 0; ks < ksteps; ks += 2) {
            step(0);
            put(a1, b1, 1, ks + 1);
            fetch(a1, b1, ks + 3);
            __syncthreads();
            step(1);
            put(a0, b0, 0, ks + 2);
            fetch(a0, b0, ks + 4);
            __syncthreads();
        }
        best_of_listed<1, 1>(a, acc, m0, n0 + wave * 32, rows, lane);
    }
}

// Rows whose second best value is near the best: into the list, their best[] back to "none yet".  Where the split GEMM
// left the rows out (skipped), all of them.
constexpr uint32_t kNearRows = 1024; // rows a workgroup looks at before it counts: one atomic each (a wave's own cost 40 us of 230 000 rows)
__global__ __launch_bounds__(256) void near_ties_kernel(NearTiesArgs a)
{
    __shared__ uint32_t s_wave[4], s_at;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, last = a.among ? *a.n_among : a.last;
    const bool all = a.skipped && *a.skipped > a.skip_from;
    for (uint32_t i0 = a.first + blockIdx.x * kNearRows; i0 < last; i0 += gridDim.x * kNearRows) {
        constexpr uint32_t kEach = kNearRows / 256u;
        uint32_t row[kEach], count = 0;
        bool near[kEach];
#pragma unroll
        for (uint32_t u = 0; u < kEach; ++u) {
            const uint32_t i = i0 + u * 256u + tid;
            row[u] = i < last ? (a.among ? a.among[i] : i) : 0u;
            near[u] = i < last;
        }
#pragma unroll
        for (uint32_t u = 0; u < kEach; ++u) {
            if (!near[u]) continue;
            const uint32_t r = row[u];
            near[u] = all || near_tie(a.best[r], a.second[r], near_margin(a.ld, a.metric, a.qnorm[r], __uint_as_float(*a.cmax)), a.metric);
            count += near[u];
        }
        uint32_t upto = count; // of this thread and the lanes before it
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(upto, off);
            if (lane >= (uint32_t)off) upto += y;
        }
        if (lane == 63u) s_wave[wave] = upto;
        __syncthreads();
        if (tid == 0) {
            const uint32_t sum = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
            s_at = sum ? atomicAdd(a.nlisted, sum) : 0u;
            if (a.also && sum) atomicAdd(a.also, sum);
        }
        __syncthreads();
        uint32_t at = s_at + upto - count;
        for (uint32_t w = 0; w < wave; ++w) at += s_wave[w];
#pragma unroll
        for (uint32_t u = 0; u < kEach; ++u) {
            if (!near[u]) continue;
            a.list[at++] = row[u];
            a.best[row[u]] = ~0ull;
            a.second[row[u]] = 0xffffffffu;
        }
        __syncthreads(); // (s_wave, s_at: read before the next round writes them)
    }
}

// What the products of the first halfs leave undecided.  Rows with two candidates (most of them): both fp32 scores by 16 lanes,
// whose sum is closer to the exact one than the fp32 kernel's; further apart than near_margin, or of lists that are
// the same bit for bit, they settle the row, else the fp32 kernel does.  Rows with more candidates go on to the products of
// the whole values (a.list), as do all rows where the first halfs were left out.
// Bound by latency: a pair is 3 rows of 4 ld bytes out of the caches.  229 376 rows x 768 with some 24 000 pairs 45 us; with a
// wave per pair 77 us instead of 24 where rows are short (200 000 x 128, a third of them pairs).
template <int RAW>
__global__ __launch_bounds__(256) void pair_ties_kernel(NearTiesArgs a)
{
    __shared__ uint32_t s_row[256], s_redo[256], s_wave[8], s_at, s_redos;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const bool all = (a.skipped && *a.skipped > a.skip_from) || (a.skipped2 && *a.skipped2 > a.skip_from2);
    for (uint32_t i0 = a.first + blockIdx.x * 256u; i0 < a.last; i0 += gridDim.x * 256u) {
        const uint32_t row = i0 + tid;
        bool many = row < a.last, pair = false;
        if (many && !all) {
            const unsigned long long best = a.best[row], next = a.next[row];
            const uint32_t third = a.second[row];
            const float margin = first_margin(a.ld, a.metric, a.qnorm[row], __uint_as_float(*a.cmax), a.left[row], __uint_as_float(*a.cmax_left));
            const float v = value_of((uint32_t)(best >> 32), a.metric);
            auto near = [&](uint32_t key) { return key != 0xffffffffu && !(fabsf(value_of(key, a.metric) - v) > margin); };
            const bool told = margin < INFINITY; // (else nothing is known of the row)
            many = !told || near(third);
            pair = !many && near((uint32_t)(next >> 32));
        }
        const unsigned long long mp = __ballot(pair), mm = __ballot(many), below = (1ull << lane) - 1ull;
        if (lane == 0u) {
            s_wave[wave] = (uint32_t)__popcll(mp);
            s_wave[4 + wave] = (uint32_t)__popcll(mm);
        }
        if (tid == 0) s_redos = 0u;
        __syncthreads();
        uint32_t pairs = 0, rest = 0, at_pair = (uint32_t)__popcll(mp & below), at_many = (uint32_t)__popcll(mm & below);
        for (uint32_t w = 0; w < 4; ++w) {
            at_pair += w < wave ? s_wave[w] : 0u;
            at_many += w < wave ? s_wave[4 + w] : 0u;
            pairs += s_wave[w];
            rest += s_wave[4 + w];
        }
        if (pair) s_row[at_pair] = row;
        if (tid == 0 && rest) s_at = atomicAdd(a.nlisted, rest);
        __syncthreads();
        if (many) {
            a.list[s_at + at_many] = row;
            a.best[row] = ~0ull;
            a.second[row] = 0xffffffffu;
        }
        const uint32_t sub = tid & 15u;
        for (uint32_t p0 = wave * 4u; p0 < pairs; p0 += 16u) { // a pair by 16 lanes
            const uint32_t p = p0 + (lane >> 4), r = s_row[p < pairs ? p : p0];
            const uint32_t c1 = (uint32_t)a.best[r], c2 = (uint32_t)a.next[r];
            const float *const x = a.x + (size_t)r * a.d, *const y1 = a.cent + (size_t)c1 * a.ld, *const y2 = a.cent + (size_t)c2 * a.ld;
            float s1 = 0.f, s2 = 0.f;
            uint32_t differ = 0;
#pragma unroll 4
            for (int i = (int)sub * 4; i < a.ld; i += 64) {
                const f32x4 w1 = *reinterpret_cast<const f32x4 *>(y1 + i), w2 = *reinterpret_cast<const f32x4 *>(y2 + i);
                const f32x4 v = dense_zeros<RAW>(dense_load<RAW>(x, i, a.d), i, a.d);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    s1 = fmaf(v[j], w1[j], s1);
                    s2 = fmaf(v[j], w2[j], s2);
                    differ |= __float_as_uint(w1[j]) ^ __float_as_uint(w2[j]);
                }
            }
            for (int off = 8; off > 0; off >>= 1) {
                s1 += __shfl_xor(s1, off);
                s2 += __shfl_xor(s2, off);
                differ |= (uint32_t)__shfl_xor((int)differ, off);
            }
            const float qn = a.qnorm[r];
            if (a.metric == PK_METRIC_L2) {
                s1 = a.cnorm[c1] - 2.f * s1 + qn;
                s2 = a.cnorm[c2] - 2.f * s2 + qn;
            }
            if (sub == 0u && p < pairs) {
                const bool same = differ == 0u, first = same ? c1 < c2 : a.metric == PK_METRIC_L2 ? s1 < s2 : s1 > s2;
                if (same || fabsf(s1 - s2) > near_margin(a.ld, a.metric, qn, __uint_as_float(*a.cmax)))
                    a.best[r] = ((unsigned long long)order_bits(first ? s1 : s2, a.metric) << 32) | (first ? c1 : c2);
                else
                    s_redo[atomicAdd(&s_redos, 1u)] = r;
            }
        }
        __syncthreads();
        const uint32_t redos = s_redos;
        if (tid == 0 && redos) {
            s_at = atomicAdd(a.nredo, redos);
            if (a.also) atomicAdd(a.also, redos);
        }
        __syncthreads();
        if (tid < redos) {
            a.redo[s_at + tid] = s_redo[tid];
            a.best[s_redo[tid]] = ~0ull;
        }
        __syncthreads(); // (the lists in LDS: read before the next round writes them)
    }
}

hipError_t launch_pair_ties(const NearTiesArgs &a, int num_cu, hipStream_t s)
{
    if (a.last <= a.first) return hipSuccess;
    if (a.ld % 64 != 0 || a.d > a.ld || a.d < 1 || a.among || !a.next || !a.left || !a.cmax_left || !a.x || !a.cent || !a.redo || !a.nredo) return hipErrorInvalidValue;
    const dim3 grid(std::min((a.last - a.first + 255u) / 256u, 8u * (uint32_t)num_cu));
    for_raw(raw_kind(a.x, a.d), [&](auto raw) { hipLaunchKernelGGL(pair_ties_kernel<raw()>, grid, dim3(256), 0, s, a); });
    return hipGetLastError();
}

hipError_t launch_near_ties(const NearTiesArgs &a, int num_cu, hipStream_t s)
{
    if (a.last <= a.first) return hipSuccess;
    if (a.ld % 64 != 0 || (a.among && (a.first != 0 || !a.n_among))) return hipErrorInvalidValue;
    hipLaunchKernelGGL(near_ties_kernel, dim3(std::min((a.last - a.first + kNearRows - 1u) / kNearRows, 4u * (uint32_t)num_cu)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_gemm_listed(GemmArgs a, int num_cu, hipStream_t s)
{
    if (a.ld % 64 != 0 || a.d > a.ld || a.d < 1 || !a.best || !a.list || !a.nlisted) return hipErrorInvalidValue;
    a.many = 6u * (uint32_t)num_cu;
    for_raw(raw_kind(a.q, a.d), [&](auto raw) {
        hipLaunchKernelGGL(gemm_listed_kernel<raw()>, dim3(3 * num_cu), dim3(256), 0, s, a);
        hipLaunchKernelGGL((gemm_scores_kernel<true, raw()>), dim3(2 * num_cu), dim3(256), 0, s, a);
    });
    return hipGetLastError();
}

} // namespace pk
