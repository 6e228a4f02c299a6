// Random permutation, permuted CSR construction, vector permutes, scans,
// row-length bins and value conversion for gfx950 (wave64).
//
// The random permutation (Section 3; Eq. 1) is the stable ascending order of
// 64-bit SplitMix64 keys. Because the keys are a pure function of the index,
// they are never stored. Up to 8192 indices are one workgroup's. Up to 8.4M, an
// LDS radix pass buckets the indices by the top 6 to 12 key bits (per-workgroup
// LDS histograms, a scan, an LDS-cursor scatter of 4-byte indices), about 256 to
// a bucket up to 128K indices and 2K beyond, and one workgroup per bucket
// sorts it in LDS (split by the next 8 bits, then a rank by (key, index) inside
// sub-buckets of ~8). Larger ranges bucket by up to 20 top bits with
// device atomics instead of LDS histograms and sort the buckets the same way.
// Either way two light passes over 4-byte indices replace the eight read-write
// passes of an LSD radix sort over 12-byte (key, index) pairs.
#include "device_common.h"
#include "internal.h"

namespace mxe {

namespace {

constexpr int kBlock = 256;
constexpr int kScanItems = 8;                          // per thread
constexpr int kScanTile = kBlock * kScanItems;         // 2048 per workgroup
constexpr int kRowsInFlight = 4;                       // rows a lane of k_gather_rows loads together

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

inline int grid_for(int64_t n, int per_block = kBlock, int64_t cap = 1 << 20) {
    int64_t g = cdiv(n, per_block);
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

// ---- fills -------------------------------------------------------------------

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_iota_i32(int32_t *p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = (int32_t)i;
}

// ---- block-level exclusive scan of one int per thread ----------------------

__device__ inline int32_t block_exclusive_scan(int32_t v, int32_t *wsum, int32_t *total) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    int32_t inc = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        int32_t t = __shfl_up(inc, off);
        if (lane >= off) inc += t;
    }
    if (lane == kWave - 1) wsum[wave] = inc;
    __syncthreads();
    int32_t woff = 0, tot = 0;
    for (int w = 0; w < kBlock / kWave; ++w) {
        if (w < wave) woff += wsum[w];
        tot += wsum[w];
    }
    __syncthreads();
    if (total) *total = tot;
    return inc - v + woff;
}

// ---- exclusive scan -----------------------------------------------------------
// Of n entries; the last one is never read (no result holds it), so a caller
// that wants the total behind its counts leaves that place unset.

__global__ __launch_bounds__(kBlock) void k_scan_tile_sums(const int32_t *in, int64_t n,
                                                           int32_t *sums) {
    __shared__ int32_t wsum[kBlock / kWave];
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    int32_t acc = 0;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        int64_t i = base + t * kBlock + threadIdx.x;
        if (i + 1 < n) acc += in[i];
    }
    int32_t tot;
    block_exclusive_scan(acc, wsum, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// The lengths of permuted rows and, a workgroup a tile of the scan, their sums:
// the scan's first pass. Bound by the random reads of rp (22.6 us with 2M rows,
// as the lengths alone took).
__global__ __launch_bounds__(kBlock) void k_perm_row_len(int32_t nrows, const int32_t *__restrict__ rp,
                                                         const int32_t *__restrict__ rperm,
                                                         int32_t *__restrict__ len, int32_t *zero,
                                                         int32_t *__restrict__ sums) {
    __shared__ int32_t wsum[kBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x == 0 && zero) *zero = 0;
    int32_t src[kScanItems], l[kScanItems], acc = 0;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) src[t] = base + t * kBlock < nrows ? rperm[base + t * kBlock] : -1;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) l[t] = src[t] >= 0 ? rp[src[t] + 1] - rp[src[t]] : 0;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        if (src[t] >= 0) len[base + t * kBlock] = l[t];
        acc += l[t];
    }
    int32_t tot;
    block_exclusive_scan(acc, wsum, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// One workgroup scans the tile sums in place (exclusive).
__global__ __launch_bounds__(kBlock) void k_scan_sums(int32_t *sums, int64_t ntiles) {
    __shared__ int32_t wsum[kBlock / kWave];
    int32_t carry = 0;
    for (int64_t base = 0; base < ntiles; base += kBlock) {
        int64_t i = base + threadIdx.x;
        int32_t v = i < ntiles ? sums[i] : 0;
        int32_t tot;
        int32_t ex = block_exclusive_scan(v, wsum, &tot);
        if (i < ntiles) sums[i] = carry + ex;
        carry += tot;
    }
}

// SCANNED: sums holds what stands before each tile; else the tiles' own sums,
// and a workgroup adds up those before its tile.
template <bool SCANNED>
__global__ __launch_bounds__(kBlock) void k_scan_tiles(const int32_t *in, int32_t *out,
                                                       int64_t n, const int32_t *sums) {
    __shared__ int32_t tile[kScanTile];
    __shared__ int32_t wsum[kBlock / kWave];
    int64_t base = (int64_t)blockIdx.x * kScanTile;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        int64_t i = base + t * kBlock + threadIdx.x;
        tile[t * kBlock + threadIdx.x] = i + 1 < n ? in[i] : 0;
    }
    int32_t before = 0;
    if constexpr (SCANNED) {
        before = sums[blockIdx.x];
    } else {
        int32_t part = 0;
        for (int i = threadIdx.x; i < (int)blockIdx.x; i += kBlock) part += sums[i];
        block_exclusive_scan(part, wsum, &before);
    }
    __syncthreads();
    int32_t loc[kScanItems];
    int32_t acc = 0;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        loc[t] = acc;
        acc += tile[threadIdx.x * kScanItems + t];
    }
    int32_t ex = block_exclusive_scan(acc, wsum, nullptr) + before;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) tile[threadIdx.x * kScanItems + t] = loc[t] + ex;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        int64_t i = base + t * kBlock + threadIdx.x;
        if (i < n) out[i] = tile[t * kBlock + threadIdx.x];
    }
}

// ---- random permutation: global bucketing (above 8.4M indices) ---------------

inline int bucket_bits(int64_t n) {          // mean bucket <= 2048 up to 2^31 indices
    int b = 0;
    while (b < 20 && (n >> b) > 2048) ++b;
    return b;
}

__device__ inline uint32_t bucket_of(uint64_t key, int bits) {
    return bits == 0 ? 0u : (uint32_t)(key >> (64 - bits));
}

__global__ __launch_bounds__(kBlock) void k_bucket_count(int64_t n, uint64_t seed, int bits,
                                                         int32_t *counts, int32_t *slot) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t b = bucket_of(sm64_key(seed, (uint64_t)i), bits);
        slot[i] = atomicAdd(&counts[b], 1);
    }
}

__global__ __launch_bounds__(kBlock) void k_bucket_scatter(int64_t n, uint64_t seed, int bits,
                                                           const int32_t *offsets,
                                                           const int32_t *slot, int32_t *items) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t b = bucket_of(sm64_key(seed, (uint64_t)i), bits);
        items[offsets[b] + slot[i]] = (int32_t)i;
    }
}

// LDS radix path (n up to kLdsPermMax): keys are bucketed by their top
// `bits` bits with per-workgroup LDS histograms (no device-wide atomics), then
// one workgroup per bucket splits it by the next kSubBits bits in LDS and
// ranks every item by (key, index) inside its sub-bucket, a handful of items.
// A range of up to kPermSmall indices is one workgroup's, split by 10 bits.
// A launch takes several permutations at once (blockIdx.y, or blockIdx.x for the
// small ones): a matrix's rows and columns, the parts of its gradient shuffles.
constexpr int kPermMaxBits = 12;                         // at most 4096 buckets
constexpr int kPermMeanBucket = 2048;
constexpr int kBucketCap = 4096;                         // items a workgroup sorts in LDS
constexpr int kSubBits = 8;                              // sub-buckets = kBlock
constexpr int64_t kLdsPermMax = (int64_t)kPermMeanBucket << kPermMaxBits;
// up to this many indices, buckets of 256 and 1024 indices to a bucketing
// workgroup, beyond it 2048 and 8192: with the latter 100K indices would keep
// 64 workgroups busy, 1.5M the count tables of the former
constexpr int64_t kPermFew = 128 * 1024;
constexpr int kPermSmall = 8192;
constexpr int kSmallBlock = 1024;
constexpr int kPermJobs = 4;

struct PermJob {
    int64_t n;
    uint64_t seed;
    int32_t *perm, *inv;                                 // inv may be null
    int32_t bits, nwg, chunk;                            // buckets' bits, workgroups and indices of each
    int32_t base;                                        // indices of the jobs before (the scan's start)
    int32_t *counts, *items;
};
struct PermJobs {
    PermJob j[kPermJobs];
};

inline int radix_bits(int64_t n) {
    const int64_t mean = n <= kPermFew ? 256 : kPermMeanBucket;
    int b = 0;
    while (b < kPermMaxBits && (n >> b) > mean) ++b;
    return b;
}

__device__ inline uint32_t top_digit(uint64_t key, int bits) {
    return bits == 0 ? 0u : (uint32_t)(key >> (64 - bits));
}
__device__ inline uint32_t sub_digit(uint64_t key, int bits) {
    return (uint32_t)(key >> (64 - bits - kSubBits)) & ((1u << kSubBits) - 1u);
}

// counts[d * nwg + w] = items of workgroup w's index range in bucket d
__global__ __launch_bounds__(kBlock) void k_perm_count(PermJobs jobs) {
    extern __shared__ int32_t hist[];
    const PermJob &J = jobs.j[blockIdx.y];
    if ((int)blockIdx.x >= J.nwg) return;
    const int nd = 1 << J.bits;
    for (int d = threadIdx.x; d < nd; d += kBlock) hist[d] = 0;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * J.chunk;
    const int64_t i1 = std::min<int64_t>(i0 + J.chunk, J.n);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kBlock)
        atomicAdd(&hist[top_digit(sm64_key(J.seed, (uint64_t)i), J.bits)], 1);
    __syncthreads();
    for (int d = threadIdx.x; d < nd; d += kBlock) J.counts[(int64_t)d * J.nwg + blockIdx.x] = hist[d];
}

// counts now hold their exclusive scan over all jobs; items[pos] = index, in
// any order inside a bucket (the bucket sort fixes the order)
__global__ __launch_bounds__(kBlock) void k_perm_scatter(PermJobs jobs) {
    extern __shared__ int32_t cursor[];
    const PermJob &J = jobs.j[blockIdx.y];
    if ((int)blockIdx.x >= J.nwg) return;
    const int nd = 1 << J.bits;
    for (int d = threadIdx.x; d < nd; d += kBlock)
        cursor[d] = J.counts[(int64_t)d * J.nwg + blockIdx.x] - J.base;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * J.chunk;
    const int64_t i1 = std::min<int64_t>(i0 + J.chunk, J.n);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kBlock) {
        const int32_t pos = atomicAdd(&cursor[top_digit(sm64_key(J.seed, (uint64_t)i), J.bits)], 1);
        J.items[pos] = (int32_t)i;
    }
}

__device__ inline bool key_less(uint64_t ka, int32_t ia, uint64_t kb, int32_t ib) {
    return ka < kb || (ka == kb && ia < ib);
}

// One workgroup per bucket: final position of each item = bucket start +
// start of its sub-bucket + its rank by (key, index) inside the sub-bucket.
// A bucket above kBucketCap (not expected from uniform keys) is ranked
// against the whole bucket in memory instead.
// Bucket d starts at counts[d * nwg] - base and ends where the next one starts.
__global__ __launch_bounds__(kBlock) void k_perm_bucket_sort(PermJobs jobs) {
    __shared__ uint64_t skey[kBucketCap];
    __shared__ int32_t sidx[kBucketCap];
    __shared__ int32_t sub[kBlock + 1];
    __shared__ int32_t cursor[kBlock];
    __shared__ int32_t wsum[kBlock / kWave];
    const PermJob &J = jobs.j[blockIdx.y];
    const int32_t d = blockIdx.x, bits = J.bits;
    if (d >= 1 << bits) return;
    const uint64_t seed = J.seed;
    const int32_t *items = J.items;
    int32_t *perm = J.perm, *inv = J.inv;
    const int32_t o = J.counts[(int64_t)d * J.nwg] - J.base;
    const int32_t m = (d + 1 < 1 << bits ? J.counts[(int64_t)(d + 1) * J.nwg] - J.base : (int32_t)J.n) - o;
    if (m > kBucketCap) {
        for (int32_t t = threadIdx.x; t < m; t += kBlock) {
            const int32_t idx = items[o + t];
            const uint64_t key = sm64_key(seed, (uint64_t)idx);
            int32_t r = 0;
            for (int32_t u = 0; u < m; ++u) {
                const int32_t iu = items[o + u];
                r += key_less(sm64_key(seed, (uint64_t)iu), iu, key, idx);
            }
            perm[o + r] = idx;
            if (inv) inv[idx] = o + r;
        }
        return;
    }
    sub[threadIdx.x] = 0;
    __syncthreads();
    for (int32_t t = threadIdx.x; t < m; t += kBlock)
        atomicAdd(&sub[sub_digit(sm64_key(seed, (uint64_t)items[o + t]), bits)], 1);
    __syncthreads();
    int32_t total;
    const int32_t ex = block_exclusive_scan(sub[threadIdx.x], wsum, &total);
    sub[threadIdx.x] = ex;
    cursor[threadIdx.x] = ex;
    if (threadIdx.x == 0) sub[kBlock] = total;
    __syncthreads();
    for (int32_t t = threadIdx.x; t < m; t += kBlock) {
        const int32_t idx = items[o + t];
        const uint64_t key = sm64_key(seed, (uint64_t)idx);
        const int32_t p = atomicAdd(&cursor[sub_digit(key, bits)], 1);
        skey[p] = key;
        sidx[p] = idx;
    }
    __syncthreads();
    for (int32_t p = threadIdx.x; p < m; p += kBlock) {
        const uint64_t key = skey[p];
        const int32_t idx = sidx[p];
        const uint32_t sd = sub_digit(key, bits);
        const int32_t b0 = sub[sd], b1 = sub[sd + 1];
        int32_t r = 0;
        for (int32_t q = b0; q < b1; ++q) r += key_less(skey[q], sidx[q], key, idx);
        perm[o + b0 + r] = idx;
        if (inv) inv[idx] = o + b0 + r;
    }
}

// exclusive scan of one int per thread of kSmallBlock threads
__device__ inline int32_t small_exclusive_scan(int32_t v, int32_t *wsum) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    int32_t inc = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int32_t t = __shfl_up(inc, off);
        if (lane >= off) inc += t;
    }
    if (lane == kWave - 1) wsum[wave] = inc;
    __syncthreads();
    int32_t woff = 0;
    for (int w = 0; w < wave; ++w) woff += wsum[w];
    return inc - v + woff;
}

// Up to kPermSmall indices by one workgroup: 4096 indices, rows and columns at
// once, take one launch where the passes above took twelve.
__global__ __launch_bounds__(kSmallBlock) void k_perm_small(PermJobs jobs) {
    __shared__ uint64_t skey[kPermSmall];
    __shared__ uint16_t sidx[kPermSmall];
    __shared__ int32_t sub[kSmallBlock + 1], cursor[kSmallBlock];
    __shared__ int32_t wsum[kSmallBlock / kWave];
    constexpr int kPer = kPermSmall / kSmallBlock, kShift = 64 - 10;
    const PermJob &J = jobs.j[blockIdx.x];
    const int t = threadIdx.x, n = (int)J.n;
    sub[t] = 0;
    __syncthreads();
    uint64_t key[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        key[k] = sm64_key(J.seed, (uint64_t)(t + k * kSmallBlock));
        if (t + k * kSmallBlock < n) atomicAdd(&sub[key[k] >> kShift], 1);
    }
    __syncthreads();
    const int32_t ex = small_exclusive_scan(sub[t], wsum);
    sub[t] = ex;                                          // each thread's own counter
    cursor[t] = ex;
    if (t == 0) sub[kSmallBlock] = n;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        if (t + k * kSmallBlock < n) {
            const int32_t p = atomicAdd(&cursor[key[k] >> kShift], 1);
            skey[p] = key[k];
            sidx[p] = (uint16_t)(t + k * kSmallBlock);
        }
    __syncthreads();
    for (int p = t; p < n; p += kSmallBlock) {
        const uint64_t kp = skey[p];
        const int32_t idx = sidx[p], d = (int32_t)(kp >> kShift);
        int32_t r = sub[d];
        for (int32_t q = sub[d]; q < sub[d + 1]; ++q) r += key_less(skey[q], sidx[q], kp, idx);
        J.perm[r] = idx;
        if (J.inv) J.inv[idx] = r;
    }
}

// ---- permuted CSR --------------------------------------------------------------

// Permuted row starts of up to kPermSmall rows by one workgroup: one launch
// where the lengths and their scan take four.
__global__ __launch_bounds__(kSmallBlock) void k_perm_row_ptr_small(int32_t nrows, const int32_t *__restrict__ rp,
                                                                    const int32_t *__restrict__ rperm,
                                                                    int32_t *__restrict__ rp_b) {
    constexpr int kPer = kPermSmall / kSmallBlock;
    __shared__ int32_t len[kPermSmall];
    __shared__ int32_t wsum[kSmallBlock / kWave];
    const int t = threadIdx.x;
    int32_t src[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) src[k] = t + k * kSmallBlock < nrows ? rperm[t + k * kSmallBlock] : -1;
#pragma unroll
    for (int k = 0; k < kPer; ++k) len[t + k * kSmallBlock] = src[k] >= 0 ? rp[src[k] + 1] - rp[src[k]] : 0;
    __syncthreads();
    int32_t v[kPer], sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        v[k] = len[t * kPer + k];
        sum += v[k];
    }
    int32_t at = small_exclusive_scan(sum, wsum);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (t * kPer + k <= nrows) rp_b[t * kPer + k] = at;
        at += v[k];
    }
    if (nrows == kPermSmall && t == kSmallBlock - 1) rp_b[nrows] = at;
}

constexpr int kSortRows = 16;                           // rows of A per wavefront, at most
constexpr int64_t kSortFew = 128 * 1024;                // rows below which a wavefront takes half of that
constexpr int kSortStage = 512;                         // staged entries per wavefront
constexpr int kSortPairs = 32;                          // rows up to this long are ranked pair by pair
constexpr int kSortLong = 2 * kSortStage;               // longest row staged alone
constexpr int kSortWaves = kBlock / kWave;

__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Each wavefront moves ROWS consecutive rows of A (row i goes to row
// rinv[i] of B, at rp_b[rinv[i]]), as many of them at a time as kSortStage
// entries hold: it stages their relabelled columns (j -> cinv[j]) in LDS, then
// every lane takes entries, finds each one's row by binary search over the
// staged row starts, and writes it at its rank among its row's new columns
// (distinct, so the rank is its sorted position). Reads stream through A in
// order, so a matrix whose columns cluster by row keeps its cinv lookups in
// cache. Short rows are ranked pair by pair. Where a row is longer than
// kSortPairs, the rows are sorted by counting: a row of L entries has L
// counters, an entry's is the one at c / ncols of them, so that after a random
// column permutation most hold one entry and a rank takes a few steps instead
// of L. A band of 10,000 rows of 256 entries in 1M rows of 8 made the kernel
// take 885 us when its wavefronts ranked them pair by pair; 2M rows of 10 FP64
// entries take 284 us either way. A row longer than the stage is ranked pair by pair, from LDS up to kSortLong
// entries, else against cinv in memory.
// A group of rows that overfills the stage is left to k_sort_deferred where
// `deferred` is given: its count, then the groups.
struct SortShared {
    int32_t buffer[kSortWaves][kSortLong];
    uint32_t counts[kSortWaves][kSortStage / 2];
    int32_t rstart[kSortWaves][kSortRows + 1];              // row starts, relative to e0
    int32_t rdest[kSortWaves][kSortRows];                   // where each row goes in B
};
template <typename V>
__device__ __attribute__((always_inline)) inline void sort_rows(
    SortShared &sh, int64_t r0, int nr, float inv_ncols, const int32_t *__restrict__ rp,
    const int32_t *__restrict__ col, const V *__restrict__ val, const int32_t *__restrict__ rinv,
    const int32_t *__restrict__ cinv, const int32_t *__restrict__ rp_b, int32_t *__restrict__ col_b,
    V *__restrict__ val_b, int32_t *__restrict__ deferred) {
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int32_t e0 = rp[r0];
    int32_t *stage = sh.buffer[wave];
    uint32_t *cnt = sh.counts[wave];
    const int32_t *rs = sh.rstart[wave];
    int32_t *rdest = sh.rdest[wave];
    const int32_t start = lane <= nr ? rp[r0 + lane] - e0 : 0;
    if (deferred && __shfl(start, nr) > kSortStage) {
        if (lane == 0) deferred[1 + atomicAdd(deferred, 1)] = (int32_t)(r0 / kSortRows);
        return;
    }
    if (lane <= nr) sh.rstart[wave][lane] = start;
    if (lane < nr) rdest[lane] = rp_b[rinv[r0 + lane]];
    wave_sync();
    auto relabel = [&](int32_t j) { return cinv ? cinv[j] : j; };
    for (int j0 = 0, j1; j0 < nr; j0 = j1) {            // rows [j0, j1): at most kSortStage entries
        const int32_t b0 = rs[j0];
        const uint64_t fit = __ballot(lane > j0 && lane <= nr && start - b0 <= kSortStage);
        if (fit == 0) {                                 // a row longer than the stage
            j1 = j0 + 1;
            const int32_t b = e0 + b0, len = rs[j1] - b0, d0 = rdest[j0];
            const bool staged = len <= kSortLong;
            if (staged)
                for (int32_t t = lane; t < len; t += kWave) stage[t] = relabel(col[b + t]);
            wave_sync();
            for (int32_t t = lane; t < len; t += kWave) {
                const int32_t c = staged ? stage[t] : relabel(col[b + t]);
                int32_t r = t;                          // rows only: order unchanged
                if (cinv) {
                    r = 0;
                    if (staged) {
                        for (int32_t u = 0; u < len; ++u) r += stage[u] < c;
                    } else {
                        for (int32_t u = 0; u < len; ++u) r += cinv[col[b + u]] < c;
                    }
                }
                col_b[d0 + r] = c;
                val_b[d0 + r] = val[b + t];
            }
            wave_sync();
            continue;
        }
        j1 = 63 - __builtin_clzll(fit);
        const int32_t n = rs[j1] - b0;
        const bool longer = __ballot(lane > j0 && lane <= j1 && start - rs[max(lane - 1, 0)] > kSortPairs) != 0;
        auto row_of = [&](int32_t i) {                  // last row of the group whose start is <= i
            int lo = j0, hi = j1 - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (rs[mid] - b0 <= i) lo = mid;
                else hi = mid - 1;
            }
            return lo;
        };
        if (!cinv || !longer) {
            for (int32_t i = lane; i < n; i += kWave) stage[i] = relabel(col[e0 + b0 + i]);
            wave_sync();
            for (int32_t i = lane; i < n; i += kWave) {
                const int j = row_of(i);
                const int32_t b = rs[j] - b0, e = rs[j + 1] - b0;
                const int32_t c = stage[i];
                int32_t r = i - b;                      // rows only: order unchanged
                if (cinv) {
                    r = 0;
                    for (int32_t u = b; u < e; ++u) r += stage[u] < c;
                }
                col_b[rdest[j] + r] = c;
                val_b[rdest[j] + r] = val[e0 + b0 + i];
            }
            wave_sync();
            continue;
        }
        // two counters to a word; after the last pass a counter holds its bucket's end
        constexpr int kPer = kSortStage / kWave;
        for (int32_t i = lane; i < kSortStage / 2; i += kWave) cnt[i] = 0;
        int32_t c[kPer];
        uint32_t at[kPer];                              // row of the group << 16 | counter
#pragma unroll
        for (int k = 0; k < kPer; ++k) c[k] = lane + k * kWave < n ? col[e0 + b0 + lane + k * kWave] : 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) c[k] = cinv[c[k]];
        wave_sync();
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int32_t i = lane + k * kWave;
            if (i >= n) continue;
            const int j = row_of(i);
            const int32_t b = rs[j], len = rs[j + 1] - b;
            // rounding keeps the order of the products, hence of the counters
            const uint32_t q = (uint32_t)(b - b0 + min((int32_t)((float)c[k] * inv_ncols * (float)len), len - 1));
            at[k] = (uint32_t)j << 16 | q;
            atomicAdd(&cnt[q >> 1], 1u << (q & 1) * 16);
        }
        wave_sync();
        uint32_t v[kSortStage / 2 / kWave], sum = 0;    // counts to starts
#pragma unroll
        for (int k = 0; k < kSortStage / 2 / kWave; ++k) {
            v[k] = cnt[lane * (kSortStage / 2 / kWave) + k];
            sum += (v[k] & 0xffffu) + (v[k] >> 16);
        }
        uint32_t inc = sum;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t t = __shfl_up(inc, o);
            if (lane >= o) inc += t;
        }
        inc -= sum;
#pragma unroll
        for (int k = 0; k < kSortStage / 2 / kWave; ++k) {
            cnt[lane * (kSortStage / 2 / kWave) + k] = inc | (inc + (v[k] & 0xffffu)) << 16;
            inc += (v[k] & 0xffffu) + (v[k] >> 16);
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const uint32_t q = at[k] & 0xffffu;
            if (lane + k * kWave < n)
                stage[atomicAdd(&cnt[q >> 1], 1u << (q & 1) * 16) >> (q & 1) * 16 & 0xffffu] = c[k];
        }
        wave_sync();
        const uint16_t *end = reinterpret_cast<const uint16_t *>(cnt);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int32_t i = lane + k * kWave;
            if (i >= n) continue;
            const int j = at[k] >> 16;
            const uint32_t q = at[k] & 0xffffu;
            const int32_t first = q ? end[q - 1] : 0, past = end[q];
            int32_t r = first;
            for (int32_t u = first; u < past; ++u) r += stage[u] < c[k];
            const int32_t d = rdest[j] - (rs[j] - b0) + r;
            col_b[d] = c[k];
            val_b[d] = val[e0 + b0 + i];
        }
        wave_sync();
    }
}

template <typename V, int ROWS>
__global__ __launch_bounds__(kBlock, 8) void k_gather_relabel_sort(
    int32_t nrows, float inv_ncols, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const V *__restrict__ val, const int32_t *__restrict__ rinv, const int32_t *__restrict__ cinv,
    const int32_t *__restrict__ rp_b, int32_t *__restrict__ col_b, V *__restrict__ val_b,
    int32_t *__restrict__ deferred) {
    __shared__ SortShared sh;
    const int64_t r0 = ((int64_t)blockIdx.x * kSortWaves + threadIdx.x / kWave) * ROWS;
    if (r0 >= nrows) return;                            // uniform per wavefront
    sort_rows<V>(sh, r0, (int)std::min<int64_t>(ROWS, nrows - r0), inv_ncols, rp, col, val, rinv, cinv, rp_b, col_b,
                 val_b, deferred);
}

// The groups left out, kDeferredRows rows to a wavefront: a band of long rows is
// a few groups among many, whose wavefronts would still be moving sixteen of
// them when all others have ended (the band above: 178 us in one launch, 110 +
// 43 in two; a launch that finds no group takes 3).
constexpr int kDeferredRows = 2, kDeferredGrid = 512;
template <typename V>
__global__ __launch_bounds__(kBlock, 8) void k_sort_deferred(
    int32_t nrows, float inv_ncols, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const V *__restrict__ val, const int32_t *__restrict__ rinv, const int32_t *__restrict__ cinv,
    const int32_t *__restrict__ rp_b, int32_t *__restrict__ col_b, V *__restrict__ val_b,
    const int32_t *__restrict__ deferred) {
    __shared__ SortShared sh;
    constexpr int kUnits = kSortRows / kDeferredRows;
    const int64_t units = (int64_t)deferred[0] * kUnits;
    for (int64_t u = blockIdx.x * (int64_t)kSortWaves + threadIdx.x / kWave; u < units;
         u += (int64_t)gridDim.x * kSortWaves) {        // uniform per wavefront
        const int64_t r0 = (int64_t)deferred[1 + u / kUnits] * kSortRows + u % kUnits * kDeferredRows;
        if (r0 < nrows)
            sort_rows<V>(sh, r0, (int)std::min<int64_t>(kDeferredRows, nrows - r0), inv_ncols, rp, col, val, rinv,
                         cinv, rp_b, col_b, val_b, nullptr);
    }
}

// ---- vector permutes (Eq. 1) -----------------------------------------------------

// Xp row j = X row perm[j], rows of c pieces of type P (leading dimensions in
// pieces). Bound by the lines the random rows pull through the L2s: 2^lsh
// lanes share a row, so a row is one request per line, and a lane carries
// kRowsInFlight rows at a time. 1.16M rows of 8 FP32 values take 40 us where
// one lane per row, value by value, took 173; 600K rows of 16 FP64 values 46
// against 262. Rows of one piece stay at 35 us (2M FP64): 2M lines of 128
// bytes, 7.3 TB/s.
template <typename P>
__global__ __launch_bounds__(kBlock) void k_gather_rows(int64_t n, int64_t c, int lsh,
                                                        const int32_t *__restrict__ perm,
                                                        const P *__restrict__ X, int64_t ldx,
                                                        P *__restrict__ Xp, int64_t ldxp) {
    const int64_t t = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    const int64_t step = ((int64_t)gridDim.x * kBlock) >> lsh;
    const int64_t q0 = t & ((1 << lsh) - 1);
    for (int64_t j = t >> lsh; j < n; j += kRowsInFlight * step) {
        int64_t src[kRowsInFlight];
#pragma unroll
        for (int u = 0; u < kRowsInFlight; ++u) src[u] = j + u * step < n ? perm[j + u * step] * ldx : -1;
        for (int64_t q = q0; q < c; q += 1 << lsh) {
            P v[kRowsInFlight];
#pragma unroll
            for (int u = 0; u < kRowsInFlight; ++u)
                if (src[u] >= 0) v[u] = X[src[u] + q];
#pragma unroll
            for (int u = 0; u < kRowsInFlight; ++u)
                if (src[u] >= 0) Xp[(j + u * step) * ldxp + q] = v[u];
        }
    }
}

// Y row perm[i] = Yp row i, rows of one piece.
template <typename P>
__global__ __launch_bounds__(kBlock) void k_scatter_rows(int64_t n, const int32_t *__restrict__ perm,
                                                         const P *__restrict__ Yp, int64_t ldyp,
                                                         P *__restrict__ Y, int64_t ldy) {
    const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (i < n) Y[perm[i] * ldy] = Yp[i * ldyp];
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_copy_cols(int32_t n, int32_t k, const T *__restrict__ src,
                                                      int64_t lds, T *__restrict__ dst,
                                                      int64_t ldd) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        for (int32_t c = 0; c < k; ++c) dst[i * ldd + c] = src[i * lds + c];
}

// Several column blocks at once: entry blockIdx.y of the table copies its
// source's k columns into columns [c0, c0 + k) of its destination, rows
// [0, n); the grid's x dimension strides over the n x k elements, one per
// thread in row-major order, so neighbouring threads touch neighbouring
// addresses on both sides.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pack_cols(const PackCols *__restrict__ table) {
    const PackCols e = table[blockIdx.y];
    const T *src = as_global((const T *)e.src);
    T *dst = as_global((T *)e.dst) + e.c0;
    const int64_t total = (int64_t)e.n * e.k;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / e.k;
        const int32_t c = (int32_t)(i - r * e.k);
        dst[r * e.ldd + c] = src[r * e.lds + c];
    }
}

// ---- value conversion --------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_f64_to_f32(const double *in, float *out, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (float)in[i];                 // v_cvt_f32_f64: round to nearest even
}

__global__ __launch_bounds__(kBlock) void k_f64_to_bf16(const double *in, uint16_t *out,
                                                        int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = bf16_from_f64(in[i]);
}

// ---- row statistics and bins ------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_row_max(int32_t nrows, const int32_t *rp,
                                                    int32_t *max_len) {
    int32_t m = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nrows;
         i += (int64_t)gridDim.x * blockDim.x)
        m = max(m, rp[i + 1] - rp[i]);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off));
    if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(max_len, m);
}

__global__ __launch_bounds__(kBlock) void k_bin_count(int32_t nrows, const int32_t *rp,
                                                      int32_t *cnt, int32_t nwg) {
    __shared__ int32_t c[kNumBins];
    if (threadIdx.x < kNumBins) c[threadIdx.x] = 0;
    __syncthreads();
    int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r < nrows) atomicAdd(&c[bin_of_length(rp[r + 1] - rp[r])], 1);
    __syncthreads();
    if (threadIdx.x < kNumBins) cnt[(int64_t)threadIdx.x * nwg + blockIdx.x] = c[threadIdx.x];
}

__global__ __launch_bounds__(kBlock) void k_bin_scatter(int32_t nrows, const int32_t *rp,
                                                        const int32_t *off, int32_t nwg,
                                                        int32_t *list) {
    __shared__ int32_t wc[kBlock / kWave][kNumBins];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int b = r < nrows ? bin_of_length(rp[r + 1] - rp[r]) : -1;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    int my_rank = 0;
    for (int q = 0; q < kNumBins; ++q) {
        uint64_t m = __ballot(b == q);
        if (b == q) my_rank = __popcll(m & lt);
        if (lane == 0) wc[wave][q] = __popcll(m);
    }
    __syncthreads();
    if (b >= 0) {
        int32_t pos = off[(int64_t)b * nwg + blockIdx.x] + my_rank;
        for (int w = 0; w < wave; ++w) pos += wc[w][b];
        list[pos] = (int32_t)r;
    }
}

__global__ void k_bin_bounds(const int32_t *off, int32_t nwg, int32_t nrows, int32_t *bin_off) {
    int b = threadIdx.x;
    if (b < kNumBins) bin_off[b] = off[(int64_t)b * nwg];
    if (b == kNumBins) bin_off[b] = nrows;
}

// ---- gradient-based shuffle (Sections 5 and 8) -------------------------------------

__global__ __launch_bounds__(kBlock) void k_row_counts(int32_t nrows, const int32_t *rp,
                                                       int32_t *counts) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nrows;
         i += (int64_t)gridDim.x * blockDim.x)
        counts[i] = rp[i + 1] - rp[i];
}

__global__ __launch_bounds__(kBlock) void k_col_counts(int64_t nnz, const int32_t *col,
                                                       int32_t *counts) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&counts[col[e]], 1);
}

// Column counts of a large matrix without an atomic per entry (they run at 28
// G/s, less where columns are heavy): the entries' columns are bucketed by
// their high bits, then each bucket is counted in LDS. 10.5M entries over 1M
// columns, a quarter of them in 14K columns: 372 us with atomics, 85 us here.
constexpr int kColBlock = 512;
constexpr int kColMinBits = 12, kColMaxBits = 15;        // columns per bucket: 4096 to 32768
constexpr int kColBuckets = 1024;
constexpr int64_t kColChunk = 16384;                     // entries of a bucketing workgroup, at least
constexpr int64_t kColPiece = 32768;                     // items a workgroup counts
constexpr int kColPieces = 64;                           // workgroups that share a bucket, at most

// Runs of equal buckets among neighbouring lanes (columns ascend in a row) take
// one LDS atomic. Returns this lane's place: its run's first, from cursor, plus
// its index in the run.
__device__ inline int32_t run_place(int32_t *cursor, int32_t d, bool valid) {
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t prev = __shfl_up(d, 1);
    const bool head = valid && (lane == 0 || prev != d);
    const uint64_t heads = __ballot(head), live = __ballot(valid);
    int32_t first = 0;
    if (head) {
        const uint64_t above = lane == kWave - 1 ? 0ull : heads & (~0ull << (lane + 1));
        const int end = above ? __builtin_ctzll(above) : 64 - __builtin_clzll(live);
        first = atomicAdd(&cursor[d], end - lane);
    }
    const uint64_t upto = heads & (~0ull >> (kWave - 1 - lane));
    const int h = upto ? 63 - __builtin_clzll(upto) : 0;
    return __shfl(first, h) + lane - h;
}

// counts[d * nwg + w] = entries of workgroup w's range in bucket d
__global__ __launch_bounds__(kColBlock) void k_col_bucket_count(int64_t nnz, int64_t chunk, int bits, int nd,
                                                                const int32_t *__restrict__ col,
                                                                int32_t *__restrict__ counts) {
    __shared__ int32_t hist[kColBuckets];
    for (int d = threadIdx.x; d < nd; d += kColBlock) hist[d] = 0;
    __syncthreads();
    const int64_t a = blockIdx.x * chunk, b = std::min(a + chunk, nnz);
    for (int64_t e = a; e < b; e += kColBlock) {         // uniform per workgroup
        const bool valid = e + threadIdx.x < b;
        run_place(hist, valid ? col[e + threadIdx.x] >> bits : -1, valid);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < nd; d += kColBlock) counts[(int64_t)d * gridDim.x + blockIdx.x] = hist[d];
}

// items[place] = the column within its bucket, in any order inside a bucket
__global__ __launch_bounds__(kColBlock) void k_col_bucket_scatter(int64_t nnz, int64_t chunk, int bits, int nd,
                                                                  const int32_t *__restrict__ col,
                                                                  const int32_t *__restrict__ offsets,
                                                                  uint16_t *__restrict__ items) {
    __shared__ int32_t cursor[kColBuckets];
    for (int d = threadIdx.x; d < nd; d += kColBlock) cursor[d] = offsets[(int64_t)d * gridDim.x + blockIdx.x];
    __syncthreads();
    const int64_t a = blockIdx.x * chunk, b = std::min(a + chunk, nnz);
    for (int64_t e = a; e < b; e += kColBlock) {
        const bool valid = e + threadIdx.x < b;
        const int32_t c = valid ? col[e + threadIdx.x] : 0;
        const int32_t at = run_place(cursor, valid ? c >> bits : -1, valid);
        if (valid) items[at] = (uint16_t)(c & ((1 << bits) - 1));
    }
}

// Bucket blockIdx.x's items, shared by as many workgroups as it holds pieces;
// out is zero where they are several.
__global__ __launch_bounds__(kColBlock) void k_col_bucket_hist(int32_t n, int bits, int32_t nwg,
                                                               const int32_t *__restrict__ offsets,
                                                               const uint16_t *__restrict__ items,
                                                               int32_t *__restrict__ out) {
    extern __shared__ int32_t hist[];                    // 1 << bits
    const int64_t i0 = offsets[(int64_t)blockIdx.x * nwg], m = offsets[(int64_t)(blockIdx.x + 1) * nwg] - i0;
    const int64_t pieces = std::min<int64_t>(std::max<int64_t>((m + kColPiece - 1) / kColPiece, 1), gridDim.y);
    if (blockIdx.y >= pieces) return;
    const int32_t c0 = (int32_t)blockIdx.x << bits, w = min(1 << bits, n - c0);
    for (int c = threadIdx.x; c < w; c += kColBlock) hist[c] = 0;
    __syncthreads();
    const int64_t a = i0 + m * blockIdx.y / pieces, b = i0 + m * (blockIdx.y + 1) / pieces;
    for (int64_t i = a + threadIdx.x; i < b; i += kColBlock) atomicAdd(&hist[items[i]], 1);
    __syncthreads();
    for (int c = threadIdx.x; c < w; c += kColBlock) {
        if (pieces == 1) out[c0 + c] = hist[c];
        else if (hist[c]) atomicAdd(&out[c0 + c], hist[c]);
    }
}

struct ArgMax { int64_t g; int64_t i; };

__device__ inline ArgMax better(ArgMax a, ArgMax b) {        // larger g; first index on ties
    return (b.g > a.g || (b.g == a.g && b.i < a.i)) ? b : a;
}

__device__ inline ArgMax block_argmax(ArgMax v, ArgMax *sh) {
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] = better(sh[threadIdx.x], sh[threadIdx.x + w]);
        __syncthreads();
    }
    return sh[0];
}

// one dimension's shuffle; a launch takes rows and columns together (blockIdx.y)
constexpr int kGradJobs = 2;
struct GradDim {
    int64_t n, na;
    const int32_t *counts;                               // entries per row or column
    const int32_t *parts;                                // pa, then pb
    int32_t *perm, *inv;
};
struct GradDims {
    GradDim d[kGradJobs];
};
// gradient g_i = h[i+1] - h[i], i < n - 1 (n >= 2)
__global__ __launch_bounds__(kBlock) void k_grad_argmax_partial(GradDims dims, ArgMax *part) {
    __shared__ ArgMax sh[kBlock];
    const int64_t n = dims.d[blockIdx.y].n;
    const int32_t *h = dims.d[blockIdx.y].counts;
    ArgMax best{INT64_MIN, INT64_MAX};
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n - 1;
         i += (int64_t)gridDim.x * blockDim.x)
        best = better(best, ArgMax{(int64_t)h[i + 1] - h[i], i});
    best = block_argmax(best, sh);
    if (threadIdx.x == 0) part[blockIdx.y * gridDim.x + blockIdx.x] = best;
}

__global__ __launch_bounds__(kBlock) void k_grad_argmax_final(int32_t nparts, const ArgMax *part,
                                                              int32_t *pivot) {
    __shared__ ArgMax sh[kBlock];
    ArgMax best{INT64_MIN, INT64_MAX};
    for (int i = threadIdx.x; i < nparts; i += kBlock) best = better(best, part[(int64_t)blockIdx.x * nparts + i]);
    best = block_argmax(best, sh);
    if (threadIdx.x == 0) pivot[blockIdx.x] = (int32_t)best.i;
}

// Riffle: A (local permutation pa of [0, na)) and B (pb of [0, nb), offset
// by na) alternate while both last; the longer part's remainder follows.
// Dimension blockIdx.y.
__global__ __launch_bounds__(kBlock) void k_riffle(GradDims dims) {
    const GradDim &D = dims.d[blockIdx.y];
    const int64_t n = D.n, na = D.na, nb = n - na, m = na < nb ? na : nb;
    const int32_t *pa = D.parts, *pb = D.parts + na;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x) {
        int32_t v;
        if (t < 2 * m) v = (t & 1) ? (int32_t)(na + pb[t >> 1]) : pa[t >> 1];
        else v = na > m ? pa[m + (t - 2 * m)] : (int32_t)(na + pb[m + (t - 2 * m)]);
        D.perm[t] = v;
        D.inv[v] = (int32_t)t;
    }
}

}  // namespace

// ============================ launchers ==========================================

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, kBlock, 4096)), dim3(kBlock), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_iota_i32(int32_t *p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_iota_i32, dim3(grid_for(n, kBlock, 4096)), dim3(kBlock), 0, s, p, n);
    return hipGetLastError();
}

size_t scan_ws_bytes(int64_t n) { return align256(sizeof(int32_t) * (size_t)(cdiv(n, kScanTile) + 1)); }

// The rest of a scan whose tiles' sums are there. Up to kScanSelf tiles each
// adds up the sums before its own, which saves a launch and the pass of one
// workgroup: the three scans of a randomization took 21.6 us where they took
// 25.2 with 90K rows, 57 for 71 with 8M rows (3907 tiles), and 703 for 693 with
// 30M (14649 tiles), where the sums read by all are the larger part.
constexpr int64_t kScanSelf = 8192;
static hipError_t launch_scan_tiles(const int32_t *in, int32_t *out, int64_t n, int32_t *sums, hipStream_t s) {
    const int64_t ntiles = cdiv(n, kScanTile);
    if (ntiles <= kScanSelf) {
        hipLaunchKernelGGL(k_scan_tiles<false>, dim3(ntiles), dim3(kBlock), 0, s, in, out, n, (const int32_t *)sums);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kBlock), 0, s, sums, ntiles);
    hipLaunchKernelGGL(k_scan_tiles<true>, dim3(ntiles), dim3(kBlock), 0, s, in, out, n, (const int32_t *)sums);
    return hipGetLastError();
}

hipError_t launch_exclusive_scan(const int32_t *in, int32_t *out, int64_t n, void *ws,
                                 hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t ntiles = cdiv(n, kScanTile);
    int32_t *sums = (int32_t *)ws;
    hipLaunchKernelGGL(k_scan_tile_sums, dim3(ntiles), dim3(kBlock), 0, s, in, n, sums);
    return launch_scan_tiles(in, out, n, sums, s);
}

namespace {

// The jobs of the LDS radix path among `count` requests, laid out in ws (or
// with ws null only measured); *small the ones of a single workgroup.
struct PermPlan {
    PermJobs mid, small;
    int nmid = 0, nsmall = 0;
    int64_t ncounts = 0;
    size_t bytes = 0;
    int max_bits = 0, max_nwg = 0;
};
PermPlan perm_plan(const PermRequest *req, int count, void *ws) {
    PermPlan p{};
    int64_t items = 0;
    for (int i = 0; i < count; ++i) {
        const PermRequest &r = req[i];
        if (r.n <= 0 || r.n > kLdsPermMax) continue;
        PermJob j{r.n, r.seed, r.perm, r.inv, 0, 1, 0, 0, nullptr, nullptr};
        if (r.n <= kPermSmall) {
            p.small.j[p.nsmall++] = j;
            continue;
        }
        j.bits = radix_bits(r.n);
        j.chunk = r.n <= kPermFew ? 1024 : 8192;
        j.nwg = (int32_t)cdiv(r.n, j.chunk);
        j.base = (int32_t)items;
        j.counts = (int32_t *)(uintptr_t)(sizeof(int32_t) * (size_t)p.ncounts);      // offsets, until ws is known
        j.items = (int32_t *)(uintptr_t)(sizeof(int32_t) * (size_t)items);
        p.ncounts += (int64_t)j.nwg << j.bits;
        items += r.n;
        p.max_bits = std::max(p.max_bits, (int)j.bits);
        p.max_nwg = std::max(p.max_nwg, (int)j.nwg);
        p.mid.j[p.nmid++] = j;
    }
    const size_t cb = align256(sizeof(int32_t) * (size_t)p.ncounts), ib = align256(sizeof(int32_t) * (size_t)items);
    p.bytes = p.nmid ? cb + ib + scan_ws_bytes(p.ncounts) : 0;
    for (int i = 0; i < p.nmid && ws; ++i) {
        p.mid.j[i].counts = (int32_t *)((char *)ws + (uintptr_t)p.mid.j[i].counts);
        p.mid.j[i].items = (int32_t *)((char *)ws + cb + (uintptr_t)p.mid.j[i].items);
    }
    return p;
}

size_t bucket_perm_ws_bytes(int64_t n) {                 // n > kLdsPermMax
    const int64_t nb = int64_t(1) << bucket_bits(n);
    return align256(sizeof(int32_t) * (nb + 1)) + 2 * align256(sizeof(int32_t) * (n + 1)) + scan_ws_bytes(nb + 1);
}

hipError_t launch_bucket_perm(const PermRequest &r, void *ws, hipStream_t s) {
    const int64_t n = r.n;
    const int bits = bucket_bits(n);
    const int64_t nb = int64_t(1) << bits;
    char *w = (char *)ws;
    int32_t *counts = (int32_t *)w;  w += align256(sizeof(int32_t) * (nb + 1));
    int32_t *slot = (int32_t *)w;    w += align256(sizeof(int32_t) * (n + 1));
    int32_t *items = (int32_t *)w;   w += align256(sizeof(int32_t) * (n + 1));
    void *scan_ws = w;
    hipError_t e = launch_fill_i32(counts, nb + 1, 0, s);
    if (e != hipSuccess) return e;
    const int g = grid_for(n, kBlock, 8192);
    hipLaunchKernelGGL(k_bucket_count, dim3(g), dim3(kBlock), 0, s, n, r.seed, bits, counts, slot);
    e = launch_exclusive_scan(counts, counts, nb + 1, scan_ws, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bucket_scatter, dim3(g), dim3(kBlock), 0, s, n, r.seed, bits,
                       (const int32_t *)counts, (const int32_t *)slot, items);
    PermJobs jobs{};
    jobs.j[0] = PermJob{n, r.seed, r.perm, r.inv, bits, 1, 0, 0, counts, items};
    hipLaunchKernelGGL(k_perm_bucket_sort, dim3((unsigned)nb), dim3(kBlock), 0, s, jobs);
    return hipGetLastError();
}

}  // namespace

size_t random_perms_ws_bytes(const PermRequest *req, int count) {
    size_t b = perm_plan(req, count, nullptr).bytes;
    for (int i = 0; i < count; ++i)
        if (req[i].n > kLdsPermMax) b = std::max(b, bucket_perm_ws_bytes(req[i].n));
    return b;
}

hipError_t launch_random_perms(const PermRequest *req, int count, void *ws, hipStream_t s) {
    if (count > kPermJobs) return hipErrorInvalidValue;
    hipError_t e;
    const PermPlan p = perm_plan(req, count, ws);
    if (p.nsmall) hipLaunchKernelGGL(k_perm_small, dim3(p.nsmall), dim3(kSmallBlock), 0, s, p.small);
    if (p.nmid) {
        const size_t lds = sizeof(int32_t) << p.max_bits;
        hipLaunchKernelGGL(k_perm_count, dim3(p.max_nwg, p.nmid), dim3(kBlock), lds, s, p.mid);
        int32_t *counts = p.mid.j[0].counts;
        if ((e = launch_exclusive_scan(counts, counts, p.ncounts, (char *)ws + p.bytes - scan_ws_bytes(p.ncounts),
                                       s)) != hipSuccess)
            return e;
        hipLaunchKernelGGL(k_perm_scatter, dim3(p.max_nwg, p.nmid), dim3(kBlock), lds, s, p.mid);
        hipLaunchKernelGGL(k_perm_bucket_sort, dim3(1 << p.max_bits, p.nmid), dim3(kBlock), 0, s, p.mid);
    }
    for (int i = 0; i < count; ++i)                      // one after the other, on the workspace of all
        if (req[i].n > kLdsPermMax && (e = launch_bucket_perm(req[i], ws, s)) != hipSuccess) return e;
    return hipGetLastError();
}

size_t sort_deferred_bytes(int32_t nrows) {
    return nrows < kSortFew ? 0 : align256(sizeof(int32_t) * (size_t)(cdiv(nrows, kSortRows) + 1));
}

size_t permuted_row_ptr_ws_bytes(int32_t nrows) { return scan_ws_bytes((int64_t)nrows + 1); }

hipError_t launch_permuted_row_ptr(int32_t nrows, const int32_t *rp, const int32_t *rperm,
                                   int32_t *rp_b, int32_t *deferred, void *ws, hipStream_t s) {
    if (nrows <= kPermSmall) {
        hipLaunchKernelGGL(k_perm_row_ptr_small, dim3(1), dim3(kSmallBlock), 0, s, nrows, rp, rperm, rp_b);
        return hipGetLastError();
    }
    int32_t *sums = (int32_t *)ws;
    const int64_t n = (int64_t)nrows + 1;
    hipLaunchKernelGGL(k_perm_row_len, dim3((unsigned)cdiv(n, kScanTile)), dim3(kBlock), 0, s, nrows, rp, rperm, rp_b,
                       deferred, sums);
    return launch_scan_tiles(rp_b, rp_b, n, sums, s);
}

hipError_t launch_gather_relabel_sort(int32_t nrows, int32_t ncols, const int32_t *rp, const int32_t *col,
                                      const void *val, int val_bytes, const int32_t *rinv,
                                      const int32_t *cinv, const int32_t *rp_b, int32_t *col_b,
                                      void *val_b, int32_t *deferred, hipStream_t s) {
    if (nrows <= 0) return hipSuccess;
    const float inv_n = 1.0f / (float)std::max(ncols, 1);
    // few rows leave CUs idle at kSortRows per wavefront: 4096 rows of 16 took
    // 10 us, half as many rows each 6.8; 2M rows of 10 fill the lanes better
    // with all of them (289 against 319 us)
    const bool few = nrows < kSortFew;
    const unsigned g = (unsigned)cdiv(nrows, (int64_t)(few ? kSortRows / 2 : kSortRows) * kSortWaves);
#define MXE_SORT(V, ROWS)                                                                                \
    hipLaunchKernelGGL((k_gather_relabel_sort<V, ROWS>), dim3(g), dim3(kBlock), 0, s, nrows, inv_n, rp, col, \
                       (const V *)val, rinv, cinv, rp_b, col_b, (V *)val_b, few ? nullptr : deferred)
#define MXE_SORT_FEW(V)                                                                                  \
    if (few) {                                                                                           \
        MXE_SORT(V, kSortRows / 2);                                                                      \
    } else {                                                                                             \
        MXE_SORT(V, kSortRows);                                                                          \
        if (deferred)                                                                                    \
            hipLaunchKernelGGL(k_sort_deferred<V>, dim3(kDeferredGrid), dim3(kBlock), 0, s, nrows, inv_n, rp, col, \
                               (const V *)val, rinv, cinv, rp_b, col_b, (V *)val_b, (const int32_t *)deferred);    \
    }
    switch (val_bytes) {
    case 8: MXE_SORT_FEW(uint64_t) break;
    case 4: MXE_SORT_FEW(uint32_t) break;
    case 2: MXE_SORT_FEW(uint16_t) break;
    default: return hipErrorInvalidValue;
    }
#undef MXE_SORT_FEW
#undef MXE_SORT
    return hipGetLastError();
}

namespace {

// bytes of the widest piece (16, 8 or 4) that k values on both sides are whole
// numbers of, every row of both on its boundary
int piece_bytes(int32_t k, const void *X, int64_t ldx, const void *Y, int64_t ldy, int elem_bytes) {
    const uint64_t a = (uint64_t)k * elem_bytes | (uint64_t)ldx * elem_bytes | (uint64_t)ldy * elem_bytes |
                       reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Y);
    return a % 16 == 0 ? 16 : a % 8 == 0 ? 8 : 4;
}

template <typename P>
hipError_t gather_rows(int64_t n, int32_t k, const int32_t *perm, const void *X, int64_t ldx, void *Xp,
                       int64_t ldxp, int elem_bytes, hipStream_t s) {
    const auto pieces = [&](int64_t elems) { return elems * elem_bytes / (int64_t)sizeof(P); };
    const int64_t c = pieces(k);
    int lsh = 0;                                         // lanes per row: c rounded up, at most a wavefront
    while ((1 << lsh) < c && (1 << lsh) < kWave) ++lsh;
    const int g = grid_for(cdiv(n, kRowsInFlight) << lsh);
    hipLaunchKernelGGL(k_gather_rows<P>, dim3(g), dim3(kBlock), 0, s, n, c, lsh, perm, (const P *)X, pieces(ldx),
                       (P *)Xp, pieces(ldxp));
    return hipGetLastError();
}

template <typename P>
hipError_t scatter_rows(int64_t n, const int32_t *perm, const void *Yp, int64_t ldyp, void *Y, int64_t ldy,
                        int elem_bytes, hipStream_t s) {
    const auto pieces = [&](int64_t elems) { return elems * elem_bytes / (int64_t)sizeof(P); };
    hipLaunchKernelGGL(k_scatter_rows<P>, dim3((unsigned)cdiv(n, kBlock)), dim3(kBlock), 0, s, n, perm,
                       (const P *)Yp, pieces(ldyp), (P *)Y, pieces(ldy));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gather_rows(int32_t n, int32_t k, const int32_t *perm, const void *X,
                              int64_t ldx, void *Xp, int64_t ldxp, int elem_bytes, hipStream_t s) {
    if (n <= 0 || k <= 0) return hipSuccess;
    if (elem_bytes != 8 && elem_bytes != 4) return hipErrorInvalidValue;
    switch (piece_bytes(k, X, ldx, Xp, ldxp, elem_bytes)) {
    case 16: return gather_rows<uint4>(n, k, perm, X, ldx, Xp, ldxp, elem_bytes, s);
    case 8: return gather_rows<uint2>(n, k, perm, X, ldx, Xp, ldxp, elem_bytes, s);
    default: return gather_rows<uint32_t>(n, k, perm, X, ldx, Xp, ldxp, elem_bytes, s);
    }
}

// Rows of one piece are scattered, wider ones gathered by the inverse: 2M rows
// of one FP64 value take 31 us scattered and 35 us gathered, 1.16M rows of 8
// FP32 values 44 us scattered and 41 us gathered.
hipError_t launch_scatter_rows(int32_t n, int32_t k, const int32_t *perm, const int32_t *inv, const void *Yp,
                               int64_t ldyp, void *Y, int64_t ldy, int elem_bytes, hipStream_t s) {
    if (n <= 0 || k <= 0) return hipSuccess;
    if (elem_bytes != 8 && elem_bytes != 4) return hipErrorInvalidValue;
    const int piece = piece_bytes(k, Yp, ldyp, Y, ldy, elem_bytes);
    if (k * (int64_t)elem_bytes != piece) return launch_gather_rows(n, k, inv, Yp, ldyp, Y, ldy, elem_bytes, s);
    switch (piece) {
    case 16: return scatter_rows<uint4>(n, perm, Yp, ldyp, Y, ldy, elem_bytes, s);
    case 8: return scatter_rows<uint2>(n, perm, Yp, ldyp, Y, ldy, elem_bytes, s);
    default: return scatter_rows<uint32_t>(n, perm, Yp, ldyp, Y, ldy, elem_bytes, s);
    }
}

hipError_t launch_copy_cols(int32_t n, int32_t k, const void *src, int64_t lds, void *dst,
                            int64_t ldd, int elem_bytes, hipStream_t s) {
    if (n <= 0 || k <= 0) return hipSuccess;
    const int g = grid_for(n, kBlock, 16384);
    if (elem_bytes == 8)
        hipLaunchKernelGGL(k_copy_cols<double>, dim3(g), dim3(kBlock), 0, s, n, k,
                           (const double *)src, lds, (double *)dst, ldd);
    else if (elem_bytes == 4)
        hipLaunchKernelGGL(k_copy_cols<float>, dim3(g), dim3(kBlock), 0, s, n, k,
                           (const float *)src, lds, (float *)dst, ldd);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_pack_cols(const PackCols *table, int32_t count, int32_t max_n, int elem_bytes,
                            hipStream_t s) {
    if (count <= 0 || max_n <= 0) return hipSuccess;
    // max_n rows of up to 16 columns per entry
    const dim3 grid(grid_for((int64_t)max_n * 16, kBlock, 2048), count);
    if (elem_bytes == 8)
        hipLaunchKernelGGL(k_pack_cols<double>, grid, dim3(kBlock), 0, s, table);
    else if (elem_bytes == 4)
        hipLaunchKernelGGL(k_pack_cols<float>, grid, dim3(kBlock), 0, s, table);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_convert_f64(const double *in, void *out, int64_t n, int dtype, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int g = grid_for(n, kBlock, 16384);
    if (dtype == VAL_F32)
        hipLaunchKernelGGL(k_f64_to_f32, dim3(g), dim3(kBlock), 0, s, in, (float *)out, n);
    else if (dtype == VAL_BF16)
        hipLaunchKernelGGL(k_f64_to_bf16, dim3(g), dim3(kBlock), 0, s, in, (uint16_t *)out, n);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

namespace {

// the bucketed column counts of nnz entries over n columns; false where atomics
// serve: below a million entries they take less than the five launches, and
// past 2^25 columns the buckets' counters outgrow the LDS
struct ColBuckets {
    int bits, nd;
    int64_t nwg, chunk, ncounts;
};
bool col_buckets(int64_t nnz, int64_t n, ColBuckets *c) {
    if (nnz < (1 << 20) || n > ((int64_t)kColBuckets << kColMaxBits)) return false;
    c->bits = kColMinBits;
    while (cdiv(n, int64_t(1) << c->bits) > kColBuckets) ++c->bits;
    c->nd = (int)cdiv(n, int64_t(1) << c->bits);
    c->chunk = std::max(kColChunk, cdiv(cdiv(nnz, 4096), kColBlock) * kColBlock);
    c->nwg = cdiv(nnz, c->chunk);
    c->ncounts = c->nwg * c->nd + 1;
    return true;
}

}  // namespace

size_t line_counts_ws_bytes(int64_t nnz, int64_t n) {
    ColBuckets c;
    if (!col_buckets(nnz, n, &c)) return 0;
    return align256(sizeof(int32_t) * c.ncounts) + align256(sizeof(uint16_t) * nnz) + scan_ws_bytes(c.ncounts);
}

hipError_t launch_line_counts(bool rows, int32_t nrows, int64_t nnz, const int32_t *rp,
                              const int32_t *col, int32_t n, int32_t *counts, void *ws, hipStream_t s) {
    if (rows) {
        if (nrows <= 0) return hipSuccess;
        hipLaunchKernelGGL(k_row_counts, dim3(grid_for(nrows, kBlock, 16384)), dim3(kBlock), 0, s,
                           nrows, rp, counts);
        return hipGetLastError();
    }
    hipError_t e = launch_fill_i32(counts, n, 0, s);
    if (e != hipSuccess || nnz <= 0) return e;
    ColBuckets c;
    if (!col_buckets(nnz, n, &c)) {
        hipLaunchKernelGGL(k_col_counts, dim3(grid_for(nnz, kBlock, 16384)), dim3(kBlock), 0, s, nnz,
                           col, counts);
        return hipGetLastError();
    }
    char *w = (char *)ws;
    int32_t *off = (int32_t *)w;     w += align256(sizeof(int32_t) * c.ncounts);
    uint16_t *items = (uint16_t *)w; w += align256(sizeof(uint16_t) * nnz);
    hipLaunchKernelGGL(k_col_bucket_count, dim3((unsigned)c.nwg), dim3(kColBlock), 0, s, nnz, c.chunk, c.bits,
                       c.nd, col, off);
    if ((e = launch_exclusive_scan(off, off, c.ncounts, w, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_col_bucket_scatter, dim3((unsigned)c.nwg), dim3(kColBlock), 0, s, nnz, c.chunk, c.bits,
                       c.nd, col, (const int32_t *)off, items);
    hipLaunchKernelGGL(k_col_bucket_hist, dim3(c.nd, kColPieces), dim3(kColBlock), sizeof(int32_t) << c.bits, s, n,
                       c.bits, (int32_t)c.nwg, (const int32_t *)off, (const uint16_t *)items, counts);
    return hipGetLastError();
}

namespace {
constexpr int kArgParts = 1024;
}

namespace {
// [partial maxima | the parts' permutations, dimension by dimension | the permutations' own workspace]
size_t grad_parts_bytes(const GradRequest *req, int count) {
    size_t b = 0;
    for (int i = 0; i < count; ++i) b += align256(sizeof(int32_t) * (size_t)(req[i].n + 1));
    return b;
}
constexpr size_t kArgBytes = (sizeof(ArgMax) * kArgParts * kGradJobs + 255) / 256 * 256;
}  // namespace

size_t gradient_perms_ws_bytes(const GradRequest *req, int count) {
    // the pivots may lie anywhere: each part as large as the whole, on either
    // path, and with the count table of a part of few indices, whose workgroups
    // and buckets are smaller
    PermRequest p[2 * kGradJobs] = {};
    for (int i = 0; i < 2 * count; ++i) p[i].n = std::max<int64_t>(req[i / 2].n, 1);
    size_t w = random_perms_ws_bytes(p, 2 * count);
    for (int i = 0; i < 2 * count; ++i) p[i].n = std::min<int64_t>(p[i].n, kLdsPermMax);
    w = std::max(w, random_perms_ws_bytes(p, 2 * count));
    PermRequest few = {kPermFew, 0, nullptr, nullptr};
    w += 2 * count * random_perms_ws_bytes(&few, 1);
    return kArgBytes + grad_parts_bytes(req, count) + w;
}

hipError_t launch_gradient_perms(const GradRequest *req, int count, int32_t *pivots, void *ws, hipStream_t s) {
    if (count > kGradJobs) return hipErrorInvalidValue;
    hipError_t e;
    ArgMax *part = (ArgMax *)ws;
    char *w = (char *)ws + kArgBytes;
    GradDims dims{};
    PermRequest parts[2 * kGradJobs];
    int nd = 0;
    int64_t n_max = 0;
    for (int i = 0; i < count; ++i) {
        if (req[i].n < 2) {                              // nothing to cut
            if ((e = launch_iota_i32(req[i].perm, req[i].n, s)) != hipSuccess ||
                (e = launch_iota_i32(req[i].inv, req[i].n, s)) != hipSuccess)
                return e;
            continue;
        }
        dims.d[nd] = GradDim{req[i].n, 0, req[i].counts, (const int32_t *)w, req[i].perm, req[i].inv};
        parts[2 * nd].seed = req[i].seed;
        w += align256(sizeof(int32_t) * (size_t)(req[i].n + 1));
        n_max = std::max(n_max, req[i].n);
        ++nd;
    }
    if (nd == 0) return hipSuccess;
    const int g = grid_for(n_max - 1, kBlock, kArgParts);
    hipLaunchKernelGGL(k_grad_argmax_partial, dim3(g, nd), dim3(kBlock), 0, s, dims, part);
    hipLaunchKernelGGL(k_grad_argmax_final, dim3(nd), dim3(kBlock), 0, s, g, (const ArgMax *)part, pivots);
    if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(s)) != hipSuccess) return e;
    for (int i = 0; i < nd; ++i) {                       // the pivots size the parts
        GradDim &D = dims.d[i];
        D.na = (int64_t)pivots[i] + 1;
        int32_t *pab = const_cast<int32_t *>(D.parts);
        const uint64_t seed = parts[2 * i].seed;
        parts[2 * i] = PermRequest{D.na, seed, pab, nullptr};
        // part B's keys continue the stream at index na: key(s, na + i) = key(s + na*gamma, i)
        parts[2 * i + 1] = PermRequest{D.n - D.na, seed + (uint64_t)D.na * 0x9e3779b97f4a7c15ull, pab + D.na, nullptr};
    }
    if ((e = launch_random_perms(parts, 2 * nd, w, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_riffle, dim3(grid_for(n_max, kBlock, 16384), nd), dim3(kBlock), 0, s, dims);
    return hipGetLastError();
}

hipError_t launch_row_max(int32_t nrows, const int32_t *rp, int32_t *max_len, hipStream_t s) {
    hipError_t e = launch_fill_i32(max_len, 1, 0, s);
    if (e != hipSuccess || nrows <= 0) return e;
    hipLaunchKernelGGL(k_row_max, dim3(grid_for(nrows, kBlock, 2048)), dim3(kBlock), 0, s, nrows,
                       rp, max_len);
    return hipGetLastError();
}

size_t row_bins_ws_bytes(int32_t nrows) {
    int64_t nwg = cdiv(nrows, kBlock);
    int64_t n = kNumBins * nwg;
    return align256(sizeof(int32_t) * (n + 1)) + scan_ws_bytes(n);
}

hipError_t launch_row_bins(int32_t nrows, const int32_t *rp, int32_t *list, int32_t *bin_off,
                           void *ws, hipStream_t s) {
    const int32_t nwg = (int32_t)cdiv(nrows, kBlock);
    if (nrows <= 0) {
        hipError_t e = launch_fill_i32(bin_off, kNumBins + 1, 0, s);
        return e;
    }
    int32_t *cnt = (int32_t *)ws;
    void *scan_ws = (char *)ws + align256(sizeof(int32_t) * ((int64_t)kNumBins * nwg + 1));
    hipLaunchKernelGGL(k_bin_count, dim3(nwg), dim3(kBlock), 0, s, nrows, rp, cnt, nwg);
    hipError_t e = launch_exclusive_scan(cnt, cnt, (int64_t)kNumBins * nwg, scan_ws, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bin_scatter, dim3(nwg), dim3(kBlock), 0, s, nrows, rp,
                       (const int32_t *)cnt, nwg, list);
    hipLaunchKernelGGL(k_bin_bounds, dim3(1), dim3(kWave), 0, s, (const int32_t *)cnt, nwg, nrows,
                       bin_off);
    return hipGetLastError();
}

}  // namespace mxe
