// Internal declarations shared by the translation units of libpancake (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <atomic>
#include <stddef.h>
#include <stdint.h>

#include "pancake.h"

// Development builds (-DPK_DEV_TIMING) record the wall clock of workgroup 0's first thread at marked
// points of a kernel; a release build holds none of this.
#ifdef PK_DEV_TIMING
#define PK_DEV_MARKS(name)                                                                      \
    static __device__ unsigned long long name##_marks[64];                                      \
    extern "C" int pk_dev_##name##_marks(unsigned long long *out)                              \
    {                                                                                           \
        return (int)hipMemcpyFromSymbol(out, HIP_SYMBOL(name##_marks), sizeof(name##_marks));   \
    }
#define PK_MARK(name, i)                                                                        \
    do {                                                                                        \
        if (blockIdx.x == 0 && threadIdx.x == 0) name##_marks[i] = wall_clock64();              \
    } while (0)
// (mark by the first thread of whichever workgroup `cond` picks)
#define PK_MARK_IF(name, i, cond)                                                               \
    do {                                                                                        \
        if ((cond) && threadIdx.x == 0) name##_marks[i] = wall_clock64();                       \
    } while (0)
#else
#define PK_DEV_MARKS(name)
#define PK_MARK(name, i) do { } while (0)
#define PK_MARK_IF(name, i, cond) do { } while (0)
#endif

namespace pk {

// ------------------------------------------------------------------ constants
constexpr int kWave = 64;
constexpr int kScanThreads = 256;     // 4 waves per workgroup in the scan kernel
constexpr int kRrTileRows = 128;      // rows per tile of the rows-in-registers scan kernel
constexpr int kRrSlots = 512;         // most query slots per tile of that kernel
constexpr int kRowBlock = 32;         // rows one wave scores per pass (two 16-wide MFMA tiles)
constexpr int kIterBytes = 256;       // bytes of one row consumed per inner iteration
constexpr int kQPadBytes = 16;        // LDS row padding of the query tile (bank spread)
constexpr int kCentroidPad = 32;      // the centroid table is zero padded to a multiple of this many rows
constexpr int kSelThreads = 256;
constexpr int kSelVec = 4;            // candidates per thread per round
constexpr int kSelCap = 4096;         // LDS key buffer of the select kernels (K + one round <= cap)
constexpr int kSelChunk = 32768;      // candidates per (query, chunk) workgroup (large batches; small ones cut finer)
constexpr unsigned long long kMaxKey = ~0ull;
constexpr int kHistBins = 64;         // per-query key histogram that tightens the emission threshold

constexpr int kErrPages = 1, kErrListFull = 2, kErrWorklist = 4;

// One arena = npages pages: vectors | norms | ids, each indexed by the local page number.
struct Arena {
    uint32_t first_page, npages;
    char *vec;       // [npages][P][row_bytes]
    float *norm;     // [npages][P]
    int64_t *ids;    // [npages][P]
};

// Device-resident description of one index (lives at the start of its first arena).
struct DevIndex {
    const float *cent;   // [nlist_pad][dpad32] fp32 centroid table, zero padded
    const float *cnorm;  // [nlist_pad] squared norms (L2 only, else zeros)
    uint32_t *list_len;  // [nlist] vectors per list
    uint32_t *main_base; // [nlist] first page of the build-time extent
    uint32_t *main_pages;// [nlist] pages in that extent
    uint32_t *dtab;      // [nlist][max_dp] delta page numbers
    uint32_t *ctr;       // [0] next free page, [1] sticky error flags, [2] pages total
    unsigned long long *stats; // running sums: [0] rows of distinct probed lists, [1] candidates, [2] tiles, [3] emitted,
                               // [4] queries whose emission region overflowed; [5] most candidates one query emitted
    int32_t nlist, nlist_pad, d, dpad32, P, max_dp, metric, storage;
    int32_t row_bytes;   // padded bytes of one stored row
    int32_t n_arenas;
    Arena arenas[PK_MAX_ARENAS];
};

__device__ __forceinline__ const Arena &arena_of(const DevIndex &ix, uint32_t page)
{
    int a = 0;
    while (a + 1 < ix.n_arenas && page >= ix.arenas[a].first_page + ix.arenas[a].npages) ++a;
    return ix.arenas[a];
}

// physical page of logical page `lp` of list `l`
__device__ __forceinline__ uint32_t phys_page(const DevIndex &ix, uint32_t l, uint32_t lp)
{
    uint32_t mp = ix.main_pages[l];
    return lp < mp ? ix.main_base[l] + lp : ix.dtab[(size_t)l * ix.max_dp + (lp - mp)];
}

// A value as an unsigned key whose ascending order is best-first (smaller = better) under
// the metric; exact inverse below.  Padding (-inf for inner product, +inf for L2) maps to
// 0xff800000 under both metrics; finite values map below it.
__device__ __forceinline__ uint32_t order_bits(float v, int metric)
{
    const uint32_t b = __float_as_uint(v);
    const uint32_t asc = b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
    return metric == PK_METRIC_L2 ? asc : ~asc;
}

__device__ __forceinline__ float value_of(uint32_t ob, int metric)
{
    const uint32_t asc = metric == PK_METRIC_L2 ? ob : ~ob;
    const uint32_t b = (asc & 0x80000000u) ? (asc ^ 0x80000000u) : ~asc;
    return __uint_as_float(b);
}

constexpr uint32_t kWorstBits = 0xff800000u;

// Bucket of a value on a per-query scale: the distance of the value from the best sampled
// value `lo`, in units of 1/inv, cut into kHistBins-1 equal buckets; everything past the
// sampled range lands in the last bucket.  Monotone in the value (each float operation
// involved is), better values get lower buckets, so "bucket <= b" is a valid cut wherever
// k candidates are known to have bucket <= b.
__device__ __forceinline__ uint32_t bucket_of(float v, float lo, float inv, int metric)
{
    float off = metric == PK_METRIC_L2 ? v - lo : lo - v;
    off = fmaxf(off, 0.f);
    const float t = fminf(off * inv, (float)(kHistBins - 1));
    return (uint32_t)t;
}

// ---- MFMA operand helpers shared by the scan kernels and the exact per-query rescoring
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Pointers taken out of a tile descriptor are generic pointers to the compiler, and loads
// through them would be flat loads: those count on the LDS counter as well, so a wait for
// an LDS read would also wait for the rows being prefetched.  These types say "global".
typedef const char __attribute__((address_space(1))) *gbytes;
typedef const float __attribute__((address_space(1))) *gfloats;
typedef const u32x4 __attribute__((address_space(1))) *gvec4;
__device__ __forceinline__ gbytes in_global(const char *p) { return (gbytes)p; }
__device__ __forceinline__ gfloats in_global(const float *p) { return (gfloats)p; }

// Rows are fetched a whole 128-byte line at a time: two loads cover 8 rows x 128 bytes each (lane l: row l & 7, 16-byte
// piece (l >> 4) + 4 * ((l >> 3) & 1)), and two moves within 16 lanes then put the pieces where MFMA wants them
// (lane l: row l & 15, piece l >> 4, of the first 64 bytes in a and of the second in b).  That is for the rows' sake that
// are read once, by non-temporal loads: a bare loop of loads over pages of 1536-byte rows, two workgroups per CU,
// reads 6.2 TB/s either way with ordinary loads, 5.1 with non-temporal loads of half a line each (the other half is
// fetched again) and 6.4 - 6.8 with non-temporal loads of whole lines (3072 bytes: 6.0, 5.5, 6.5; 4096: 5.8, 5.7, 6.2).
__device__ __forceinline__ void line_to_operands(u32x4 &a, u32x4 &b)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int x = (int)a[d], y = (int)b[d];
        a[d] = (uint32_t)__builtin_amdgcn_update_dpp(x, y, 0x128, 0xf, 0xc, false); // lanes 8 .. 15 of 16: y's lanes 0 .. 7
        b[d] = (uint32_t)__builtin_amdgcn_update_dpp(y, x, 0x128, 0xf, 0x3, false); // lanes 0 .. 7: x's lanes 8 .. 15
    }
}

// How a kernel reads rows of d floats of the caller's: not at all (padded copies), in aligned 16-byte pieces (kRawVec: d a
// multiple of 4), in 16-byte pieces that begin anywhere (any_load), or, where a row has less than one of these, float by float.
enum { kRawNot, kRawVec, kRawAny, kRawShort };
inline int raw_kind(const float *rows, int d)
{
    return d < 4 ? kRawShort : (d & 3) == 0 && (reinterpret_cast<uintptr_t>(rows) & 15) == 0 ? kRawVec : kRawAny;
}

// Four floats of a dense row of d (four at least) from column `col` on, of a row that begins anywhere: the load, unconditional, from the
// row's last four floats where fewer are left, and what the columns hold, zeros past the row's end.  In two parts, as
// arranging them waits for the load.  (A load of 16 bytes wants no more than the alignment of its elements.)
struct __attribute__((packed, aligned(4))) AnyFour {
    u32x4 v;
};
__device__ __forceinline__ u32x4 any_load(const uint32_t *row, int col, int d)
{
    return reinterpret_cast<const AnyFour *>(row + (col + 4 <= d ? col : d - 4))->v;
}
__device__ __forceinline__ u32x4 any_zeros(u32x4 v, int col, int d)
{
    const int past = col + 4 - d; // how far the load was moved; all of it past the end from 4 on
    u32x4 r = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int s = 0; s + j < 4; ++s) r[j] = (s == 0 ? past <= 0 : past == s) ? v[j + s] : r[j];
    return r;
}

// The same in each of the three forms.  The loads are unconditional (past the row's end from its last floats): the compiler waits
// for a load under a condition before it issues the next.  (Nor is the form asked for while reading: a condition that is the same for all
// lanes splits the loads as well.)
template <int RAW>
__device__ __forceinline__ u32x4 raw_load(const uint32_t *row, int col, int d)
{
    static_assert(RAW == kRawVec || RAW == kRawAny || RAW == kRawShort, "");
    if constexpr (RAW == kRawVec) return *reinterpret_cast<const u32x4 *>(row + (col < d ? col : d - 4));
    else if constexpr (RAW == kRawAny) return any_load(row, col, d);
    else {
        u32x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = row[col + j < d ? col + j : d - 1];
        return v;
    }
}
template <int RAW>
__device__ __forceinline__ u32x4 raw_zeros(u32x4 v, int col, int d)
{
    if constexpr (RAW == kRawAny) return any_zeros(v, col, d);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = col + j < d ? v[j] : 0u;
    return v;
}

// 16 bytes of a query row (A) against 16 bytes of a stored row (B), fp32 accumulation: one
// v_mfma_f32_16x16x32_f16, or four v_mfma_f32_16x16x4_f32.  Every kernel that scores a
// (row, query) pair issues these in the same order over the row, so the value of a pair does
// not depend on the kernel that computed it.
template <int STORAGE>
__device__ __forceinline__ void mfma_step(f32x4 &acc, const u32x4 &qa, const u32x4 &xb)
{
    if constexpr (STORAGE == PK_F16) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, qa), __builtin_bit_cast(half8, xb),
                                                     acc, 0, 0, 0);
    } else {
        f32x4 qf = __builtin_bit_cast(f32x4, qa), xf = __builtin_bit_cast(f32x4, xb);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[0], xf[0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[1], xf[1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[2], xf[2], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[3], xf[3], acc, 0, 0, 0);
    }
}

// squared L2 distance from the inner product and the two squared norms (one expression, used
// by every kernel that returns a fine-search value)
__device__ __forceinline__ float l2_from_dot(float xn, float dot, float qn) { return fmaxf(xn - 2.f * dot + qn, 0.f); }

// exclusive scan of in[0,n) into out[0,n) by one workgroup (up to 1024 threads); returns the
// total.  A thread takes 4 consecutive elements, so 4096 elements need one round of barriers;
// out may be the same array as in.
__device__ __forceinline__ uint32_t block_exscan(const uint32_t *in, uint32_t *out, uint32_t n, uint32_t *s_wave /*[17]*/)
{
    uint32_t carry = 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    for (uint32_t base = 0; base < n; base += 4u * blockDim.x) {
        const uint32_t i = base + 4u * threadIdx.x;
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = i + j < n ? in[i + j] : 0u;
        const uint32_t t = v[0] + v[1] + v[2] + v[3];
        uint32_t x = t;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off);
            if (lane >= off) x += y;
        }
        if (lane == 63) s_wave[wave] = x;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t acc = 0;
            for (int w = 0; w < nwaves; ++w) {
                const uint32_t tw = s_wave[w];
                s_wave[w] = acc;
                acc += tw;
            }
            s_wave[16] = acc;
        }
        __syncthreads();
        uint32_t run = carry + s_wave[wave] + x - t;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (i + j < n) out[i + j] = run;
            run += v[j];
        }
        carry += s_wave[16];
        __syncthreads();
    }
    return carry;
}

// One unit of scan work: the rows of one page, or of a part of it (wl_lay_query's tiles where there are few: 64 or 32 rows from
// anywhere in the page; the rows-stationary kernels': kRrTileRows), against one group of query slots.
struct Tile {
    const char *x;    // the tile's first row
    const float *xn;  // squared norms of its rows (L2), else unused
    uint32_t row0;    // position of its first row in the list
    uint32_t qbeg;    // first slot of the group in slot_query / slot_out
    uint16_t nrows;   // its rows
    uint16_t qcnt;    // slots in the group (<= MQ); of wl_lay_query's tiles: the group's number in its list
    uint32_t list;    // of wl_lay_query's tiles: handle * nlist_max + list
};
static_assert(sizeof(Tile) == 32, "Tile is 32 bytes");

// Handles of one call, passed to kernels by value (fits the 4 KiB kernel-argument space).
struct MultiArgs {
    const DevIndex *ix[PK_MAX_HANDLES];
    uint32_t qlo[PK_MAX_HANDLES + 1];   // handle a owns query rows [qlo[a], qlo[a+1])
    int32_t n;
};

// --------------------------------------------------------------- launch APIs
// (each enqueues on `s` and returns the HIP status of the launch)

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, size_t n, hipStream_t s);
// several ranges in one launch: a launch that clears a few words takes 2 - 5 us of the stream, and as long of the host
struct FillRanges {
    static constexpr int kMost = 10;
    uint32_t *p[kMost];
    size_t n[kMost];
    uint32_t v[kMost];
    int ranges; // as many as were added; more than there is room for, and the launch refuses
    void add(void *at, uint32_t value, size_t words)
    {
        if (ranges < kMost) {
            p[ranges] = static_cast<uint32_t *>(at);
            n[ranges] = words;
            v[ranges] = value;
        }
        ++ranges;
    }
};
hipError_t launch_fill_ranges(const FillRanges &a, hipStream_t s);
hipError_t launch_copy_i32(const int32_t *src, int32_t *dst, int64_t n, hipStream_t s);

// queries -> storage type, zero padded rows, squared norms of the converted values
hipError_t launch_prep_queries(const float *q, int64_t nq, int d, int storage, int row_bytes, void *qs,
                               float *qnorm, hipStream_t s);

struct ScanArgs {
    const Tile *tiles;
    const uint32_t *ntiles;      // device scalar
    const uint32_t *batch;       // device scalar: tiles taken per grab (>= 1)
    const char *qs;              // prepared queries [nq][row_bytes]
    const float *qnorm;          // [nq]
    const uint32_t *slot_query;  // slot -> query row
    const uint32_t *slot_out;    // slot -> first output element of the (query, list) pair
    float *out;                  // dense mode: values, one per (slot, row)
    // gated mode (tau != NULL): a value is emitted only if its key is <= tau[query]; it is
    // appended as (key << 32 | position) to the query's region of cbuf
    const uint32_t *tau;         // [nq] threshold keys from the sample (never change)
    const float *tlo;            // [nq] best sample value: origin of the bucket scale
    const float *tinv;           // [nq] bucket scale (see bucket_of)
    uint32_t *hist;              // [nq][kHistBins] emitted candidates per bucket (zero before the launch)
    uint32_t *tcur;              // [nq] running bucket limit shared by all workgroups (starts at kHistBins-1)
    union { // (not side by side: a line more of arguments is 0.3 us of a search of one query)
        uint32_t ecap;           // entries of each query's region of cbuf: query q owns [q * ecap, (q + 1) * ecap)
        uint32_t slot_room;      // launch_scan_few (no regions): entries of slot_query and slot_out
    };
    uint32_t *ccnt;              // [nq] candidates that passed the gate so far (zero before the launch); those past
                                 // ecap are counted but not stored, and the query is then selected by rescoring
    unsigned long long *cbuf;
    uint32_t *tile_ctr;          // device scalar, zero before the launch: batches handed out after the first round
    int k, use_hist;
    int row_bytes, metric, storage, mq;
    uint32_t rr_first;           // rows-in-registers kernel: pairs of tiles its (first) launch starts with, one per workgroup
    bool rr_join;                // ... this launch joins one that is running (same counter, same rr_first)
    bool nt;                     // fine search: the rows are read past the caches (they would not stay in them anyway)
    // laid mode (lcnt != NULL): the tiles and slots are those of wl_lay_query, and every value is written
    const uint32_t *lcnt;        // pairs of each list (of all handles)
    uint32_t *mins;              // or null: best key of every 16 values, as they lie in `out`
    uint32_t tile_cap;           // more tiles than this: the layout was refused, nothing is scanned
    int grab_div;                // tiles per grab = tiles / (grid * this), 1 .. 8
};
hipError_t launch_scan(const ScanArgs &a, int grid, hipStream_t s);
hipError_t launch_scan_ks(const ScanArgs &a, int grid, hipStream_t s);
constexpr int kFewRows = 64; // most rows of a tile that launch_scan_few takes
hipError_t launch_scan_few(const ScanArgs &a, int grid, hipStream_t s);
hipError_t launch_scan_rr(const ScanArgs &a, int grid, hipStream_t s);
int scan_rr_lds_bytes();
int scan_lds_bytes(int row_bytes, int mq);
int scan_ks_lds_bytes(int mq);
int scan_max_mq(int row_bytes, int storage, int lds_limit);

// Tile schedule shared by the list-scan kernels.  The first tile of every workgroup is fixed (tile b for
// workgroup b); later batches come from one counter, so uneven tiles still balance while
// the launch does not start with a burst of atomics.  A batch is `grab` tiles; the first batch
// is a single tile so that the emission gates get their first refresh early.  The request for the next
// batch is issued when a batch starts and collected when it ends, and the descriptor of the
// next tile is fetched while the current tile is scored.  Every workgroup stops the first
// time it is handed a batch past the end.
struct Sched {
    uint32_t t, end, ntiles, grab;
    uint32_t nblk; // workgroups that take tiles (all of the launch, unless its first ones do other work)
    int parity;
    bool fresh; // t is the first tile of a batch
    // bid: this workgroup's number among the nblk that take tiles
    __device__ __forceinline__ void start(uint32_t nt, uint32_t g, uint32_t bid, uint32_t nb)
    {
        ntiles = nt;
        grab = g;
        nblk = nb;
        t = bid;
        end = t + 1 < nt ? t + 1 : nt;
        parity = 0;
        fresh = true;
    }
    // one thread asks for the batch after the current one (s_misc[2*parity], [2*parity+1] = start, size)
    __device__ __forceinline__ void request(const ScanArgs &a, uint32_t *s_misc, uint32_t asker = 0u) const
    {
        if (threadIdx.x == asker && nblk < ntiles) {
            // One atomic per batch and no other access to the counter: every workgroup of the
            // grid claims from this one address, and a second access per claim (a load, to
            // size the batch by what is left) measurably slows the whole scan.
            const uint32_t want = grab;
            s_misc[2 * parity] = nblk + atomicAdd(a.tile_ctr, want);
            s_misc[2 * parity + 1] = want;
        }
    }
    // index of the tile after t; at the end of a batch this collects the requested batch (block-wide)
    __device__ __forceinline__ uint32_t peek(const uint32_t *s_misc, uint32_t &next_end, bool &next_fresh) const
    {
        if (t + 1 < end) {
            next_end = end;
            next_fresh = false;
            return t + 1;
        }
        next_fresh = true;
        if (nblk >= ntiles) {
            next_end = ntiles;
            return ntiles;
        }
        __syncthreads();
        const uint32_t st = s_misc[2 * parity], sz = s_misc[2 * parity + 1];
        next_end = st + sz < ntiles ? st + sz : ntiles;
        return st;
    }
};


// Dynamic LDS beyond 64 KB has to be allowed per kernel and device.  Every scan kernel is cleared
// once per device for the most a workgroup can have, so the value never depends on the call
// that happens to come first and threads serving different handles cannot undo each other.
constexpr int kMaxDevices = 64;
struct LdsCleared {
    std::atomic<int> on[kMaxDevices];
};

// (fixed: bytes of LDS that the kernel declares itself; the two together are at most what a workgroup can have)
template <typename K>
inline hipError_t allow_lds(K kernel, LdsCleared &c, int fixed = 0)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool tracked = dev >= 0 && dev < kMaxDevices;
    if (!tracked || c.on[dev].load(std::memory_order_acquire) == 0) {
        int most = 0;
        e = hipDeviceGetAttribute(&most, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
        if (e != hipSuccess) return e;
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, most - fixed);
        if (e != hipSuccess) return e;
        if (tracked) c.on[dev].store(1, std::memory_order_release);
    }
    return hipSuccess;
}

template <typename K, typename A>
inline hipError_t launch_with_lds(K kernel, LdsCleared &c, int lds, const A &a, int grid, int threads, hipStream_t s)
{
    const hipError_t e = allow_lds(kernel, c);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, s, a);
    return hipGetLastError();
}



struct SelectArgs {
    const float *vals;            // candidate values, or NULL when keys are given
    const unsigned long long *keys; // candidate keys (value key << 32 | position)
    const uint32_t *qoff;         // [nq] first candidate of each query
    const uint32_t *qcnt;         // [nq] candidates of each query
    int metric, K, nchunks;
    int chunk;                    // candidates per (query, chunk) workgroup
    unsigned long long *partial;  // [nq][nchunks][K]
};
hipError_t launch_select_partial(const SelectArgs &a, int64_t nq, hipStream_t s);
constexpr int kMaxSamplePages = 64;      // most pages of one query's threshold sample
constexpr uint32_t kWlSmallLists = 2048; // most lists (all handles of a call) whose work list is laid out inside another kernel's launch
constexpr int kDenseSelectMax = 8192; // longest score row the register-resident selection takes

hipError_t launch_select_probes(const unsigned long long *partial, int nchunks, int K, int nprobe, int64_t nq,
                                int32_t *probes, hipStream_t s);

struct FinalArgs {
    int K, k, nprobe, metric, storage, row_bytes;
    const unsigned long long *keys;   // emitted candidates: query q owns [q * ecap, (q + 1) * ecap)
    unsigned long long *spill;        // the same regions, writable: scratch of a query that is rescored
    uint32_t ecap;
    const uint32_t *qcnt;             // [nq] candidates that passed the gate (more than ecap: region overflowed)
    const uint32_t *pair_off;         // [nq][nprobe+1] start of each probe's segment inside the query's range
    const int32_t *probes;            // [nq][nprobe]
    const uint16_t *qagent;           // [nq] handle number
    const char *qs;                   // prepared queries [nq][row_bytes] (storage type), for the rescoring
    const float *qnorm;               // [nq]
    int64_t *out_ids;
    float *out_dist;
    // Queries whose region overflowed, scored again by many workgroups (launch_rescue): the first `rregions` of them,
    // in query order, have a region of rcap keys each; rcnt[q] counts what query q got (more than rcap: overflowed again)
    unsigned long long *rkeys;
    uint32_t *rcnt;                   // [nq] zero before launch_rescue
    uint32_t rregions, rcap;          // rregions 0: launch_rescue was not called
    const uint32_t *hist;             // [nq][kHistBins] candidates the scan emitted per bucket, stored or not (null: not counted)
    const float *tlo, *tinv;          // [nq] bucket scale
    // every value of the query's range instead of emitted keys (keys is null): query q's at vals[q * width]
    const float *vals;
    const uint32_t *mins;             // best key of every 16 values: where width is more than kReadOnce
    uint32_t width;
    const uint32_t *ntiles;           // with vals: more tiles than tile_cap, and nothing was scanned
    uint32_t tile_cap;
};
constexpr uint32_t kReadOnce = 8192; // values that the workgroup of a final selection holds in registers
constexpr uint32_t kRescueCap = 4096;    // keys per rescue region: what the final selection takes in registers
constexpr uint32_t kRescueRegions = 128; // most queries of a call that are rescued
// workgroups of launch_rescue: two per CU, and one at least for every region (a device of few CUs has fewer than regions)
inline int rescue_grid(int num_cu, uint32_t regions) { return 2 * num_cu > (int)regions ? 2 * num_cu : (int)regions; }
hipError_t launch_rescue(const FinalArgs &a, const MultiArgs &m, int64_t nq, int grid, hipStream_t s);
hipError_t launch_select_final(const FinalArgs &a, const MultiArgs &m, int64_t nq, hipStream_t s);

// Per-query bookkeeping of the coarse step, filled while the queries are prepared.
struct QueryMeta {
    uint32_t stride;               // elements between the score rows of consecutive queries
    uint32_t *cand_off, *cand_cnt; // [nq] score row of each query and its length (nlist of its handle)
    uint16_t *qagent;              // [nq] handle number of each query
    uint32_t *clear;               // words the fine step wants zeroed before it starts (or null)
    uint32_t nclear;
};
// fp32 queries -> zero padded rows and squared norms, plus the bookkeeping above
hipError_t launch_prep_coarse(const float *q, int64_t nq, int d, int row_bytes, void *qs, float *qnorm,
                              const QueryMeta &meta, const MultiArgs &m, hipStream_t s);

// Centroid scoring of small query segments (16 centroids x `chunk` queries per workgroup).
struct CentroidArgs {
    const char *qs;      // prepared fp32 queries [nq][row_bytes]
    const float *qnorm;  // [nq]
    float *out;          // score of (query q, centroid c of q's handle) at out[q * stride + c]
    uint32_t stride;
    int row_bytes, metric;
    int chunk;           // queries per workgroup: 16, 32, 48 or 64
    uint32_t blk[PK_MAX_HANDLES + 1]; // first workgroup of handle a, [n] = all; a handle scored elsewhere owns none
    // Optional extras that save a launch each on small batches:
    //   meta.cand_off != null: this kernel also does the per-query bookkeeping of the coarse step and clears
    //   the words in meta.clear (qs then are the caller's own rows: no padding needed, no norms for inner product);
    //   best != null: instead of writing scores, every query keeps its best (score key << 32 | list) by
    //   atomicMin (top-1 assignment of inserts; best[] must hold ~0 on entry).
    QueryMeta meta;
    unsigned long long *best;
    //   raw (with meta): qs are the caller's dense rows of d floats; under L2 the scores are written without the query's own
    //   norm;
    //   rows, norm: the fp32 rows, zero padded to row_bytes, and their squared norms are written too; halves, half_norm: the
    //   same of the rows rounded to half precision, padded to half_bytes (each of them, or null).
    int raw, d, half_bytes;
    char *rows, *halves;
    float *norm, *half_norm;
};
hipError_t launch_centroid_scores(const CentroidArgs &a, const MultiArgs &m, hipStream_t s);
// Of the rows (of one handle) whose best two values are near, as the split GEMM left them, the best by the centroid kernel.
// (Arguments of their own: the other launches' would be a line longer, 0.3 us of a search of one query.)
struct NearRowsArgs {
    const unsigned long long *split_best; // [.] the split GEMM's best (value key << 32 | list)
    const uint32_t *second, *cmax;        // and second values; largest squared centroid norm (as bits)
    int32_t *lists;                       // [.] out: split_best's list, or kListByRedo for a row whose best is in CentroidArgs::best
    uint32_t parts;                       // (set by the launch) workgroups that share a group of 64 rows
};
// (a.best: ~0 on entry; a.qnorm is given whatever the metric)
hipError_t launch_centroid_near(CentroidArgs a, const MultiArgs &m, NearRowsArgs n, int nlist_pad, hipStream_t s);

// merge of per-handle result rows into one row per query (k <= 1024: rank fits 10 bits, handle 7)
struct UnionArgs {
    const int64_t *ids;  // [n_handles][nq][k] rows of the handles, each sorted best first, -1 padded
    const float *dist;   // [n_handles][nq][k]
    int n_handles, k, metric;
    int64_t nq;
    int32_t *out_src;    // [nq][k] position of the handle in the scope, -1 for padding
    int64_t *out_ids;    // [nq][k]
    float *out_dist;     // [nq][k]
};
hipError_t launch_union_merge(const UnionArgs &a, hipStream_t s);

// Level cascade (early termination): bookkeeping between the searches of two levels.
struct LevelArgs {
    int64_t nq;
    int k, metric, level;
    bool first, last;        // first: every query is open; last: this level ends every search
    const float *stop;       // [nq]
    uint32_t *open;          // [nq] 1 while the query has not ended (written when first)
    int32_t *level_out;      // [nq] or null
    const int64_t *row_ids;  // [nq][k] this level's rows (null when first: they are already in out_*)
    const float *row_dist;   // [nq][k]
    int64_t *out_ids;        // [nq][k]
    float *out_dist;         // [nq][k]
};
// rows of this level -> output for the open queries; closes those the rule (or the last level) ends
hipError_t launch_level_accept(const LevelArgs &a, hipStream_t s);
// probes[q][*] = -1 for queries that are no longer open (their lists are not scanned)
hipError_t launch_level_mask(int32_t *probes, int nprobe, const uint32_t *open, int64_t nq, hipStream_t s);

struct WorklistArgs {
    const int32_t *probes;     // [nq][nprobe]; entries outside [0, nlist) are ignored
    const uint16_t *qagent;    // [nq]
    int64_t nq;
    int nprobe, n_handles, nlist_max, scan_grid, scan_grid_hot, grab_div, hot_grab;
    int mq;                    // slots per group of a regular tile
    int mq_hot;                // slots per group of a hot tile
    int hot_rows;              // rows per hot tile: 0 = a page; else a divisor of the page size (rows-stationary kernel)
    uint32_t hot_from;         // lists probed by more than this many queries of the batch are hot
    uint32_t *lcnt, *lstart, *lfill, *ltile, *lhtile; // [n_handles * nlist_max]
    bool lcnt_cleared;         // the coarse step of the same search has zeroed lcnt already
    uint32_t tile_rows;        // with width: rows of a tile (a divisor of every handle's page size), or 0: a page
    uint32_t *pair_off;        // [nq][nprobe+1]
    uint32_t *ccnt;            // [nq] zeroed here (emission counters of the gated scan)
    uint32_t *slot_query, *slot_out; // [nq * nprobe]; slot_out = first position of the pair inside the query's range
    Tile *tiles, *tiles_hot;
    uint32_t tile_cap;
    uint32_t *scalars;         // [0] ntiles [1] tile counter [2] grab size
    uint32_t *scalars_hot;     // [0] hot tiles [1] tile counter [2] grab size
    // whole layout in one go (wl_lay_query), values written whole:
    uint32_t cap;              // slots of each list (the most queries of a handle)
    uint32_t width;            // elements of each query's range
    // one handle only: its list lengths, page size and list count, so that the work-list layout of a small batch
    // reads them without first chasing the handle's descriptor (null / 0 otherwise)
    const uint32_t *len1;
    uint32_t P1, nlist1;
};

// Threshold sampling: the first `sp` pages of each query's first probed list are scored
// densely; the k-th best of them bounds the query's k-th best overall.
struct SampleArgs {
    const int32_t *probes;     // [nq][nprobe]
    const uint16_t *qagent;
    int nq;
    int rescued;               // queries whose region overflows may be scored again: slot_out is cleared for that
    int nprobe, sp, k, metric, scan_grid;
    uint32_t span;             // values per query = sp * rows per page (same for all handles)
    Tile *tiles;               // [nq * sp]
    uint32_t *slot_query;      // [nq] = q
    uint32_t *slot_out;        // [nq] = q * span; with `rescued`, once the threshold exists: 0 (the query's rescue counter)
    float *vals;               // [nq][span], pre-filled with the padding value by the kernel
    uint32_t *scalars;         // [0] ntiles [1] tile counter [2] grab size
    uint32_t *tau;             // [nq] out: k-th best sample key, or 0xffffffff
    float *tlo;                // [nq] out: best sample value
    float *tinv;               // [nq] out: bucket scale = (kHistBins-1) / |k-th best (or worst) sample value - best|
    uint32_t *hist;            // [nq][kHistBins] zeroed here
    uint32_t *tcur;            // [nq] out: running bucket limit, starts at kHistBins-1
};
hipError_t launch_worklist_count(const WorklistArgs &a, const SampleArgs &sm, const MultiArgs &m, hipStream_t s);
hipError_t launch_worklist_tiles(const WorklistArgs &a, const MultiArgs &m, hipStream_t s);
// wa / ma given (small batches): the launch also builds the second half of the work list (launch_worklist_tiles is not needed)
hipError_t launch_tau(const SampleArgs &a, hipStream_t s, const WorklistArgs *wa = nullptr, const MultiArgs *ma = nullptr);
// small batches: the sample's tiles, the thresholds and the second half of the work list in one launch (in place of
// launch_scan over the sample, launch_tau and launch_worklist_tiles); sm.span at most 4096
hipError_t launch_sample_tau(const ScanArgs &a, const SampleArgs &sm, const WorklistArgs &wa, const MultiArgs &ma, int grid,
                             hipStream_t s);
// wa / sm / ma given: the selection's workgroups also do launch_worklist_count's work for their queries, or with wa->width
// the whole work list (a.slot_query and slot_out then have wa->cap entries per list, a.scalars' first two words are zero);
// add: the scores (L2) lack the query's squared norm
hipError_t launch_select_dense(const float *vals, const uint32_t *qoff, const uint32_t *qcnt, uint32_t max_cnt, int metric,
                               int K, int64_t nq, int32_t *probes, hipStream_t s, const WorklistArgs *wa = nullptr,
                               const SampleArgs *sm = nullptr, const MultiArgs *ma = nullptr, const float *add = nullptr);

// dense coarse scoring on the matrix cores (large query batches, build)
struct GemmArgs {
    const float *q;      // [m][ld] prepared fp32 queries (zero padded rows)
    const float *c;      // [n_pad][ld] centroid table
    const float *qnorm;  // [m]
    const float *cnorm;  // [n_pad]
    float *out;          // [m][stride]
    int m, n, n_pad, n_store, ld, metric;
    uint32_t stride;
    // launch_gemm_listed: q are the caller's dense rows [.][d], qnorm and best indexed by row like them
    const uint32_t *list, *nlisted; // rows to score, and how many (on the device)
    unsigned long long *best;       // [.] out: best (value key << 32 | column) of the listed rows
    int d;
    uint32_t many;                  // (set by launch_gemm_listed)
};
hipError_t launch_gemm_scores(const GemmArgs &a, hipStream_t s);
hipError_t launch_gemm_listed(GemmArgs a, int num_cu, hipStream_t s); // the same values, of listed rows: their best columns
// rows whose second best value (second[]: as the split GEMM left it) is near their best, into a list
struct NearTiesArgs {
    uint32_t first, last;        // rows [first, last) of best, second, qnorm
    const uint32_t *among, *n_among; // or (among not null) the *n_among rows in it, at most last of them; first is 0 then
    unsigned long long *best;    // of the listed rows: back to ~0,
    uint32_t *second;            //   and to all ones
    const uint32_t *cmax;
    const float *qnorm;
    const uint32_t *skipped;     // or null: more than skip_from in it and the rows are listed all, whatever best and second hold
    uint32_t skip_from;
    uint32_t *list, *nlisted, *also; // also (or null): raised as nlisted is
    int ld, metric;
    // launch_pair_ties alone (rows [first, last)): best, next and second as the products of first halfs left them; rows of more
    // than two candidates into list, pairs that fp32 sums do not settle into redo (also: raised as nredo is)
    const uint32_t *cmax_left;
    const float *left;
    const uint32_t *skipped2;    // as skipped
    uint32_t skip_from2;
    const unsigned long long *next;
    const float *x, *cent, *cnorm; // dense fp32 rows [.][d]; the table [.][ld]
    int d;
    uint32_t *redo, *nredo;
};
hipError_t launch_near_ties(const NearTiesArgs &a, int num_cu, hipStream_t s);
hipError_t launch_pair_ties(const NearTiesArgs &a, int num_cu, hipStream_t s);

// Two values of a row closer than this are told apart by the fp32 kernel.  The fp32 sum of ld products, two at a time,
// is off by about 2^-25 sqrt(ld / 2) of |x| |c| in one standard deviation (measured: 1e-6 |x|^2 between two L2 values
// at 768 elements), the split's by a third of it; 2^-21 sqrt(ld) is twenty of them.
// Squared lengths below kTinySquare have lost what makes them a bound (elements below 2^-63 leave nothing in them, while the
// scaled products of such rows still tell lists apart): nothing is further apart than that, and the fp32 kernel decides.
// Above it the squares that were lost are 2^-24 of the sum at most, whatever the row's width.
constexpr float kTinySquare = 8.07793567e-28f; // 2^-90
__device__ __forceinline__ float near_margin(int ld, int metric, float qn, float cmax)
{
    if (metric == PK_METRIC_L2 ? qn + cmax < kTinySquare : qn < kTinySquare || cmax < kTinySquare) return INFINITY;
    return 4.76837158e-7f * sqrtf((float)ld) * (metric == PK_METRIC_L2 ? qn + cmax : sqrtf(qn) * sqrtf(cmax));
}

// What two values of a row may differ by and still be in the other order for the fp32 kernel, where they are sums of the first
// halfs' products alone, <x', c'> where x = x' + x", c = c' + c": off by <x", c> + <x', c">, which is
// |x"| |c| + |x| |c"| at most (Cauchy-Schwarz; left: |x"|, cm_left: the most |c"| is; the factor covers the rounding of the
// lengths themselves).  Lengths that are no numbers, or so large that a value might not be one: nothing is further apart than that.
__device__ __forceinline__ float first_margin(int ld, int metric, float qn, float cm, float left, float cm_left)
{
    if (!(qn + cm < 1.32922800e36f)) return INFINITY; // 2^120
    const float off = 1.001f * (left * sqrtf(cm) + sqrtf(qn) * cm_left);
    return near_margin(ld, metric, qn, cm) + (metric == PK_METRIC_L2 ? 4.f : 2.f) * off; // (two products, and twice each under L2)
}

// Rows whose values cannot all be compared (a NaN among them: from a NaN or an infinity in the row or in a centroid, or
// from finite values whose products overflow) are decided by the fp32 kernel too: their second value is kNoOrder.
constexpr uint32_t kNoOrder = 0u;           // below the key of every number
constexpr uint32_t kWorstKey = 0xfffffffeu; // the most a list's key can be, so that all ones stays "no list"

// whether a row with that best (value key << 32 | column) and that second value is decided by more exact values
__device__ __forceinline__ bool near_tie(unsigned long long best, uint32_t second, float margin, int metric)
{
    if (second == kNoOrder || second == 0xffffffffu) return second == kNoOrder;
    const float gap = fabsf(value_of(second, metric) - value_of((uint32_t)(best >> 32), metric));
    return !(gap > margin);
}

// top-1 of the same products, every fp32 operand held as two halfs (see pk_gemm.hip)
struct SplitRowsArgs {
    const float *x;      // [m][d] rows, dense
    const float *c;      // [n_c][ld] centroid table, zero padded
    uint32_t m, n_c;
    int d, ld;
    char *xs, *cs;       // [m][4 * ld], [n_c][4 * ld] out: split rows (or null)
    char *xh, *ch;       // [m][2 * ld], [n_c][2 * ld] out: the first halfs alone (or null)
    float *x_back, *c_back; // [m] (or null), [n_c] out: what undoes the row's scale
    float *qnorm;        // [m] out: squared norms, or null
    float *copy;         // [m][ld] out: fp32 rows, zero padded, or null
    char *half_rows;     // [m][half_bytes] out: rows rounded to half precision, zero padded, or null
    float *half_norm;    // [m] out: their squared norms
    int half_bytes;
    unsigned long long *best; // [m] set to ~0, or null
    uint32_t *second;    // [m] set to all ones, or null
    unsigned long long *redo; // [m] set to ~0, or null
    uint32_t *cmax;      // raised to the largest squared norm of the centroids (as bits), or null
    float *left;         // [m] out: length of what the first halfs leave out of the row, or null
    uint32_t *cmax_left; // raised to the most that is of a centroid (as bits), or null
    QueryMeta meta;      // as in launch_prep_coarse (cand_off null: not wanted)
};
hipError_t launch_split_rows(const SplitRowsArgs &a, const MultiArgs &m, hipStream_t s);
struct SplitGemmArgs {
    const char *q, *c;   // split rows [m][4 * ld], [n_pad][4 * ld]; or, with `left`, first halfs [m][2 * ld], [n_pad][2 * ld]
    const float *q_back, *c_back, *qnorm, *cnorm; // (norms: L2 only)
    unsigned long long *best; // [m] best (value key << 32 | column) by atomicMin; ~0 on entry
    int m, n, n_pad, ld, metric;
    // optional: the value key of the second best column where it is near the best (else all ones, as on entry)
    uint32_t *second;         // [m] (or null: no row's near ties are of interest)
    const uint32_t *cmax;     // largest squared norm of the centroids (as bits)
    const uint32_t *skipped, *skipped2; // or null: with more than skip_from in it the launch does nothing
    uint32_t skip_from, skip_from2;
    const float *left;        // [m] or null: the products of the first halfs alone, near by first_margin
    const uint32_t *cmax_left;
    unsigned long long *next; // with left: [m] the second best (value key << 32 | column), where it is near the best (else all ones, as on
                              // entry); second[] then has a value key near the best where there are more than two such columns
    // launch_gemm_split_listed: dense fp32 rows [.][d], split on the way; best, second, q_back, qnorm indexed by row like them
    const float *x;
    const uint32_t *list, *nlisted; // rows to score, and how many (on the device)
    int d;
};
hipError_t launch_gemm_split(const SplitGemmArgs &a, int num_cu, hipStream_t s);
hipError_t launch_gemm_split_listed(const SplitGemmArgs &a, int num_cu, hipStream_t s);

// build / insert
// the lists of a top-1 assignment (low words of best[]), how many rows each list gets (cnt: zero before), and, with slots, a
// place of its own for every row among those of its list
hipError_t launch_lists_of_best(const unsigned long long *best, int64_t n, int nlist, int32_t *assign, uint32_t *cnt, uint32_t *slots, hipStream_t s);
constexpr int kLdsLists = 8192; // most lists that a workgroup counts in LDS (32 KB)
hipError_t launch_build_pages(const DevIndex *ix, const uint32_t *cnt, hipStream_t s); // main_base, main_pages, list_len and ctr[0]
hipError_t launch_build_places(const DevIndex *ix, const int32_t *assign, int64_t n, uint32_t *slots, hipStream_t s);
hipError_t launch_scatter_build(const DevIndex *ix, const float *x, const int64_t *ids, const uint32_t *rows_at, int64_t n, int64_t id0,
                                int pieces, hipStream_t s); // (pieces: of 64 elements in a stored row)
hipError_t launch_store_centroids(const float *c, int nlist, int d, int dpad32, int nlist_pad, int metric,
                                  float *cent, float *cnorm, hipStream_t s);
// Removes the rows whose id is among ids[0..m), m <= kDeleteChunk.  One pass removes at most kDeleteChunk
// rows; if more rows carry the ids (several rows under one id), the sticky flag says so and the caller
// runs the pass again.
constexpr int kDeleteChunk = 4096;
constexpr int kDeleteUnit = 1024; // rows of one list that a workgroup examines at a time
struct DeleteArgs {
    const DevIndex *ix;
    int nlist, m;
    bool first;                // first pass of the call: nothing has been counted yet
    int bits;                  // (set by launch_delete) the hash set has 1 << bits slots
    const int64_t *ids;        // [m]
    uint32_t *unit_start;      // scratch [nlist + 1] (tables of more than kLdsLists lists): units of the lists before each one
    unsigned long long *hits;  // scratch [kDeleteChunk]: (list << 32) | position of the rows to go
    uint32_t *hit_rank;        // scratch [kDeleteChunk]: per hit, the hits of its list before it,
    uint32_t *hit_cnt;         //   the hits of its list,
    uint32_t *hit_len0;        //   and, for its list's first hit, the list's length before the pass
    uint32_t *scal;            // of the handle: [0] rows found (zero between passes), [1] of them taken, [2] sticky: a pass found more than it could take
    unsigned long long *removed; // of the handle: rows removed by the call
    uint32_t *host;            // pinned [3]: rows removed (low, high word), the sticky flag
};
hipError_t launch_delete(DeleteArgs a, int num_cu, hipStream_t s);
// copies every list into the contiguous extents of `dst` (dst's tables are already in place)
// (skip: optional [dst nlist] flags of lists the caller fills itself; lists beyond src's are skipped too)
hipError_t launch_compact_pages(const DevIndex *src, const DevIndex *dst, uint32_t new_pages, const uint8_t *skip,
                                hipStream_t s);
// the first min(len, length of list l) members of list l as dense fp32 rows [.][d] and / or their ids
hipError_t launch_gather_list(const DevIndex *ix, uint32_t l, uint32_t len, float *rows, int64_t *ids, hipStream_t s);
// 2-means of every list to split, all lists in the same launches, straight from the lists' pages
// (Section 4.4: a light k-means on the device decides the split).  Job j splits list job_list[j].
constexpr int kSplitUnit = 1024; // rows of one list that a workgroup assigns at a time
struct SplitArgs {
    const DevIndex *ix;
    int njobs;
    const uint32_t *job_list;  // [njobs]
    const uint32_t *job_len;   // [njobs] members
    const uint32_t *job_unit0; // [njobs + 1] units of the jobs before each one
    const uint32_t *job_row0;  // [njobs] members of the jobs before each one: where the job's part of side[] starts
    double *cent;              // [njobs][2][d] the two centroids
    double *sum;               // [njobs][2][d] sums of the members of each side (zero between the launches)
    unsigned long long *cnt;   // [njobs][2] members of each side (zero between the launches)
    unsigned long long *cnt_out; // [njobs][2] the counts of the last assignment
    int32_t *side;             // [sum of job_len] 0 / 1 per member, by position in its list
};
// first centroids: the member with the smallest id and the member with the largest id
hipError_t launch_split_init(const SplitArgs &a, hipStream_t s);
// one Lloyd iteration: every member to the nearer centroid (ties to the first), then the centroids to the
// means of their members (a centroid without members stays)
hipError_t launch_split_iterate(const SplitArgs &a, uint32_t total_units, int d, hipStream_t s);
// the jobs' centroids into a dense fp32 table [.][d]: row job_list[j] and row nlist0 + j
hipError_t launch_split_centroids(const SplitArgs &a, int nlist0, float *dense, hipStream_t s);
// list l of src split by side[r]: side 0 stays list l of dst, side 1 becomes list lnew of dst (slot: scratch [len])
hipError_t launch_split_list(const DevIndex *src, const DevIndex *dst, uint32_t l, uint32_t lnew, const int32_t *side,
                             uint32_t *slot, uint32_t len, hipStream_t s);
// k-means update step (Lloyd): members of every cluster gathered, then one workgroup per cluster
struct KmeansArgs {
    const float *x;        // [n][d] training rows
    const int32_t *assign; // [n] cluster of each row
    int64_t n;
    int d, nlist;
    uint32_t *cnt;         // [nlist] in: members of each cluster
    uint32_t *start, *fill; // [nlist] each (scratch; fill: zeros)
    uint32_t *piece0;      // [nlist + 1] (scratch) parts of at most 256 members of the clusters before each one
    uint32_t *members;     // [n] row numbers in cluster-major order (scratch)
    float *centroids;      // [nlist][d] in: centroids the assignment used; out: means of the members
    double *sums;          // [nlist][d] scratch, zeros: per-cluster totals
    double *sq;            // [nlist] scratch, zeros: per-cluster totals of |x|^2
    double *inertia;       // one word, zero: receives the sum of squared distances of the assignment
};
hipError_t launch_kmeans_update(const KmeansArgs &a, hipStream_t s);
// Insert: slots for the vectors of every handle of the batch (one workgroup per handle; rows [qlo[a], qlo[a+1]) of
// assign / slots / assigned_out belong to handle a), then the rows.  Groups of kInsertGroup vectors of a handle are
// inserted whole or not at all.
constexpr int kInsertGroup = 1024;
// batches of at most this many vectors per handle: reservation and row writes share one launch
constexpr int kFusedAppend = 64;
struct AppendIds {
    int64_t id0[PK_MAX_HANDLES]; // first id of each handle's segment when the caller gives no ids
};
// the lists are assign[], or the low words of best[] (written to lists[]); ranks: scratch like slots
// (redo, with assign = lists: entries that are kListByRedo are the low words of redo[], and written, too)
constexpr int32_t kListByRedo = -1;
hipError_t launch_reserve(const MultiArgs &ma, const int32_t *assign, const unsigned long long *best,
                          const unsigned long long *redo, int32_t *lists, uint32_t *ranks, uint32_t *slots, int32_t *assigned_out, hipStream_t s);
hipError_t launch_append(const MultiArgs &ma, const AppendIds &idc, const float *x, const int64_t *ids,
                         const int32_t *assign, const uint32_t *slots, unsigned long long *reset, hipStream_t s);
// assign == null: the lists are the low words of best[] (left by the centroid kernel), which is reset to ~0
hipError_t launch_reserve_append(const MultiArgs &ma, const AppendIds &idc, const float *x, const int64_t *ids,
                                 const int32_t *assign, unsigned long long *best, uint32_t *slots, int32_t *assigned_out,
                                 hipStream_t s);

} // namespace pk
