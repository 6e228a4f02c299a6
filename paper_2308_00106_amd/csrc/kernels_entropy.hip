// 2D block nonzero histogram and its Shannon entropy (Section 4, Eq.
// eq:entropy; Section 5's 2D histogram view) for gfx950.
//
// Histogram: one workgroup per block-row (split further only when a block-row
// holds more than 64K entries). The block-row's entries are a contiguous
// nonzero range [row_ptr[r0], row_ptr[r1]), so the workgroup streams col_idx
// once, coalesced, and counts into an LDS copy of its G_c bins. Runs of equal
// block-column among neighbouring lanes (common in clustered matrices, whose
// sorted columns fall in the same block) are merged with one LDS atomic per
// run. A workgroup that owns its block-row writes the bins with plain stores.
//
// Entropy: H = ln S - (1/S) sum_b h_b ln h_b (nats), the same real number as
// -sum p ln p with p = h / S. Every term is evaluated in double-double (about
// 106 bits) with a fixed reduction order, so the result is deterministic; the
// final rounding to FP64 is certified against an error bound, which makes it
// the correctly rounded value of the exact entropy.
#include "device_common.h"
#include "internal.h"

#include <algorithm>

namespace mxe {

namespace {

constexpr int kBlock = 256;
constexpr int kHistLds = 16384;                 // block-columns held in LDS (at most 64 KB)
constexpr int64_t kHistSplitItems = 16384;      // entries per workgroup before splitting
constexpr int64_t kHistMinGroups = 2048;        // workgroups enough to fill the chip
constexpr int kEntGrid = 1024;                  // fixed grid: fixed reduction order

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

__global__ __launch_bounds__(kBlock) void k_zero_u32(uint32_t *p, int64_t n, uint32_t *q, int64_t nq) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n + nq;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (i < n) p[i] = 0;
        else q[i - n] = 0;
    }
}

// grid: (grid_r, split). Block-row bi covers rows [ceil(bi M / G_r), ceil((bi+1) M / G_r)).
__global__ __launch_bounds__(kBlock) void k_block_hist(int32_t nrows, int32_t ncols,
                                                       const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ col,
                                                       int32_t grid_r, int32_t grid_c,
                                                       double inv_n, uint32_t *__restrict__ hist) {
    extern __shared__ uint32_t bins[];                  // grid_c counters when they fit
    const int64_t bi = blockIdx.x;
    const int split = gridDim.y, part = blockIdx.y;
    const int64_t r0 = (bi * nrows + grid_r - 1) / grid_r;
    const int64_t r1 = ((bi + 1) * nrows + grid_r - 1) / grid_r;
    const int64_t e0 = rp[r0], e1 = rp[r1];
    const int64_t len = e1 - e0;
    const int64_t a = e0 + len * part / split, b = e0 + len * (part + 1) / split;
    const bool in_lds = grid_c <= kHistLds;
    uint32_t *out_row = hist + bi * grid_c;
    if (in_lds) {
        for (int c = threadIdx.x; c < grid_c; c += kBlock) bins[c] = 0;
        __syncthreads();
    }
    const int lane = threadIdx.x & (kWave - 1);
    // the workgroup walks [a, b) in steps of kBlock, so every wave is either
    // fully inside or partly inside a step: loop bounds are uniform per wave
    for (int64_t base = a; base < b; base += kBlock) {
        const int64_t e = base + threadIdx.x;
        const bool valid = e < b;
        const int32_t bj = valid ? block_index(col[e], grid_c, ncols, inv_n) : -1;
        if (in_lds) {
            const int32_t prev = __shfl_up(bj, 1);
            const bool head = valid && (lane == 0 || prev != bj);
            const uint64_t heads = __ballot(head);
            const uint64_t live = __ballot(valid);
            if (head) {
                const uint64_t above = lane == kWave - 1 ? 0ull : heads & (~0ull << (lane + 1));
                const int end = above ? __builtin_ctzll(above) : 64 - __builtin_clzll(live);
                atomicAdd(&bins[bj], (uint32_t)(end - lane));
            }
        } else if (valid) {
            atomicAdd(&out_row[bj], 1u);
        }
    }
    if (in_lds) {
        __syncthreads();
        if (split == 1) {
            for (int c = threadIdx.x; c < grid_c; c += kBlock) out_row[c] = bins[c];
        } else {
            for (int c = threadIdx.x; c < grid_c; c += kBlock)
                if (bins[c]) atomicAdd(&out_row[c], bins[c]);
        }
    }
}

struct EntPartial { double hi, lo; unsigned long long s, nz; };

// Sums over the workgroup's N threads, in a fixed order; the same in every thread.
template <int N> struct EntShared {
    dd acc[N];
    unsigned long long s[N], nz[N];
};
template <int N>
__device__ inline void block_reduce(dd &acc, unsigned long long &s, unsigned long long &nz, EntShared<N> &sh) {
    sh.acc[threadIdx.x] = acc;
    sh.s[threadIdx.x] = s;
    sh.nz[threadIdx.x] = nz;
    __syncthreads();
    for (int w = N / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            sh.acc[threadIdx.x] = dd_add(sh.acc[threadIdx.x], sh.acc[threadIdx.x + w]);
            sh.s[threadIdx.x] += sh.s[threadIdx.x + w];
            sh.nz[threadIdx.x] += sh.nz[threadIdx.x + w];
        }
        __syncthreads();
    }
    acc = sh.acc[0];
    s = sh.s[0];
    nz = sh.nz[0];
}

// Rounds v (absolute error <= eps) to FP64; *ok = 0 when v - eps and v + eps
// round differently (the correctly rounded value is then not certain).
__device__ inline double certified_round(dd v, double eps, int *ok) {
    double lo = v.hi + (v.lo - eps);
    double hi = v.hi + (v.lo + eps);
    if (lo != hi) *ok = 0;
    return v.hi + v.lo;
}

// From T = sum h ln h (double-double), S = sum h and the count of nonzero
// bins: result = {H bits, H nats, certified (1/0), S}, each H rounded to FP64
// and certified against the error bound (Eq. 2 with p = h / S).
__device__ inline void entropy_finish(dd acc, unsigned long long s, unsigned long long nz, double *result) {
    if (s == 0 || nz <= 1) {            // no distribution, or all mass in one bin
        result[0] = 0.0;
        result[1] = 0.0;
        result[2] = 1.0;
        result[3] = (double)s;
        return;
    }
    const double sd = (double)s;        // exact: s < 2^53
    dd ln_s = dd_ln_int(sd);
    dd mean = dd_div(acc, dd{sd, 0.0});
    dd h_nats = dd_sub(ln_s, mean);
    dd h_bits = dd_div(h_nats, kLn2);
    // error bound: every double-double step is accurate to ~2^-100 relative and
    // the reduction is ~30 levels deep; 2^-90 (ln S + 1) leaves a 2^7 margin
    const double eps = 0x1p-90 * (ln_s.hi + 1.0);
    int ok = 1;
    result[0] = certified_round(h_bits, eps * 2.0, &ok);
    result[1] = certified_round(h_nats, eps, &ok);
    result[2] = ok ? 1.0 : 0.0;
    result[3] = sd;
}

// Count of counts: cc[c] = number of bins holding exactly c entries, for
// c < kCountDirect (LDS per workgroup, then exact integer atomics into one
// table, zero at first); bins with more entries add c ln c to the workgroup's
// partial directly. S and the nonzero-bin count are summed alongside.
constexpr int kCountDirect = 4096;

__global__ __launch_bounds__(kBlock) void k_entropy_counts(const uint32_t *__restrict__ hist,
                                                           int64_t bins, uint32_t *__restrict__ cc,
                                                           EntPartial *part) {
    __shared__ uint32_t lcc[kCountDirect];
    __shared__ EntShared<kBlock> sh;
    for (int c = threadIdx.x; c < kCountDirect; c += kBlock) lcc[c] = 0;
    __syncthreads();
    dd acc{0.0, 0.0};
    unsigned long long s = 0, nz = 0;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < bins;
         i += (int64_t)gridDim.x * kBlock) {
        const uint32_t h = hist[i];
        s += h;
        nz += h != 0;
        if (h < kCountDirect) {
            if (h >= 2) atomicAdd(&lcc[h], 1u);
        } else {
            const double hd = (double)h;
            acc = dd_add(acc, dd_mul_d(dd_ln_int(hd), hd));
        }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < kCountDirect; c += kBlock)
        if (lcc[c]) atomicAdd(&cc[c], lcc[c]);
    block_reduce(acc, s, nz, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = EntPartial{acc.hi, acc.lo, s, nz};
}

// T = sum over c of cc[c] c ln c (c in fixed order per thread, then a fixed
// tree) plus the large-count partials in workgroup order. (Done by the last
// workgroup of the kernel before, it saved a launch but cost a device-wide
// fence in each: 88 us for a 1024 x 1024 grid where the two take 32.)
constexpr int kFinalBlock = 1024;
__global__ __launch_bounds__(kFinalBlock) void k_entropy_final(const uint32_t *__restrict__ cc,
                                                               const EntPartial *part, int nparts,
                                                               double *result) {
    __shared__ EntShared<kFinalBlock> sh;
    uint32_t n[kCountDirect / kFinalBlock];
#pragma unroll
    for (int k = 0; k < kCountDirect / kFinalBlock; ++k) n[k] = cc[threadIdx.x + k * kFinalBlock];
    dd acc{0.0, 0.0};
    unsigned long long s = 0, nz = 0;
    for (int i = threadIdx.x; i < nparts; i += kFinalBlock) {
        acc = dd_add(acc, dd{part[i].hi, part[i].lo});
        s += part[i].s;
        nz += part[i].nz;
    }
    for (int k = 0; k < kCountDirect / kFinalBlock; ++k) {
        const int c = threadIdx.x + k * kFinalBlock;
        if (c < 2 || n[k] == 0) continue;
        const double cd = (double)c;
        acc = dd_add(acc, dd_mul_d(dd_mul_d(dd_ln_int(cd), cd), (double)n[k]));
    }
    block_reduce(acc, s, nz, sh);
    if (threadIdx.x == 0) entropy_finish(acc, s, nz, result);
}

// Hierarchical 2D entropy (Section 5). Regions are numbered level by level,
// row-major in a level; region (a, b) of level L holds the bins r with
// floor(r * Lr / G_r) = a, i.e. r in [ceil(a G_r / Lr), ceil((a + 1) G_r / Lr)),
// and likewise columns. `parts` workgroups share each region, workgroup p
// taking cells p*kRegBlock + t, p*kRegBlock + t + parts*kRegBlock, ... of it;
// where they are several, one more per region combines them in index order.
constexpr int kRegBlock = 1024;
struct Levels { int32_t n, level[16]; };
struct Region { int32_t r0, r1, c0, c1; };

__device__ inline Region region_at(const Levels &l, int64_t index, int64_t grid_r, int64_t grid_c) {
    int i = 0;
    int64_t lr, lc;
    for (;; ++i) {
        lr = std::min<int64_t>(l.level[i], grid_r);
        lc = std::min<int64_t>(l.level[i], grid_c);
        if (index < lr * lc) break;
        index -= lr * lc;
    }
    const int64_t a = index / lc, b = index % lc;
    return Region{(int32_t)((a * grid_r + lr - 1) / lr), (int32_t)(((a + 1) * grid_r + lr - 1) / lr),
                  (int32_t)((b * grid_c + lc - 1) / lc), (int32_t)(((b + 1) * grid_c + lc - 1) / lc)};
}

__global__ __launch_bounds__(kRegBlock) void k_entropy_regions(const uint32_t *__restrict__ hist, int32_t grid_r,
                                                               int32_t grid_c, Levels levels, int32_t parts,
                                                               EntPartial *__restrict__ part,
                                                               double *__restrict__ out) {
    __shared__ EntShared<kRegBlock> sh;
    const int64_t region = blockIdx.x / parts, p = blockIdx.x % parts;
    const Region rg = region_at(levels, region, grid_r, grid_c);
    const int64_t w = rg.c1 - rg.c0, cells = (int64_t)(rg.r1 - rg.r0) * w;
    dd acc{0.0, 0.0};
    unsigned long long s = 0, nz = 0;
    for (int64_t i = p * kRegBlock + threadIdx.x; i < cells; i += (int64_t)parts * kRegBlock) {
        const uint32_t h = hist[(int64_t)(rg.r0 + i / w) * grid_c + rg.c0 + i % w];
        s += h;
        nz += h != 0;
        if (h >= 2) {
            const double hd = (double)h;
            acc = dd_add(acc, dd_mul_d(dd_ln_int(hd), hd));
        }
    }
    block_reduce(acc, s, nz, sh);
    if (threadIdx.x != 0) return;
    if (parts == 1) entropy_finish(acc, s, nz, out + 4 * region);
    else part[blockIdx.x] = EntPartial{acc.hi, acc.lo, s, nz};
}

__global__ __launch_bounds__(kWave) void k_entropy_regions_final(const EntPartial *__restrict__ part,
                                                                 int32_t parts, double *__restrict__ out) {
    __shared__ EntShared<kWave> sh;
    const EntPartial *pr = part + (int64_t)blockIdx.x * parts;
    dd acc{0.0, 0.0};
    unsigned long long s = 0, nz = 0;
    for (int i = threadIdx.x; i < parts; i += kWave) {
        acc = dd_add(acc, dd{pr[i].hi, pr[i].lo});
        s += pr[i].s;
        nz += pr[i].nz;
    }
    block_reduce(acc, s, nz, sh);
    if (threadIdx.x == 0) entropy_finish(acc, s, nz, out + 4 * (int64_t)blockIdx.x);
}

// Workgroups per region: enough that the largest region's cells are spread
// at ~4 per thread, at most 64, and about 16K workgroups in total.
int32_t region_parts(int32_t grid_r, int32_t grid_c, const int32_t *levels, int32_t nlevels,
                     int32_t nregions) {
    int64_t max_cells = 0;
    for (int32_t i = 0; i < nlevels; ++i) {
        const int64_t lr = std::min(levels[i], grid_r), lc = std::min(levels[i], grid_c);
        max_cells = std::max(max_cells, cdiv(grid_r, lr) * cdiv(grid_c, lc));
    }
    int64_t p = cdiv(max_cells, 4 * (int64_t)kRegBlock);
    p = std::min<int64_t>(p, 64);
    p = std::min<int64_t>(p, std::max<int64_t>(1, 16384 / std::max(nregions, 1)));
    return (int32_t)std::max<int64_t>(p, 1);
}

}  // namespace

hipError_t launch_block_hist(int32_t nrows, int32_t ncols, int64_t nnz, const int32_t *rp,
                             const int32_t *col, int32_t grid_r, int32_t grid_c, uint32_t *hist,
                             void *entropy_ws, hipStream_t s) {
    const int64_t bins = (int64_t)grid_r * grid_c;
    int64_t split = std::max(cdiv(cdiv(nnz, grid_r), kHistSplitItems), cdiv(kHistMinGroups, grid_r));
    if (split < 1) split = 1;
    if (split > 65535) split = 65535;
    const int64_t nz = split > 1 || grid_c > kHistLds ? bins : 0;
    const int64_t nq = entropy_ws ? kCountDirect : 0;
    if (nz + nq > 0) {
        int g = (int)std::min<int64_t>(cdiv(nz + nq, kBlock), 65536);
        hipLaunchKernelGGL(k_zero_u32, dim3(g), dim3(kBlock), 0, s, hist, nz, (uint32_t *)entropy_ws, nq);
    }
    const double inv_n = 1.0 / (double)ncols;
    const size_t lds = grid_c <= kHistLds ? sizeof(uint32_t) * (size_t)grid_c : 0;
    hipLaunchKernelGGL(k_block_hist, dim3(grid_r, (unsigned)split), dim3(kBlock), lds, s, nrows,
                       ncols, rp, col, grid_r, grid_c, inv_n, hist);
    return hipGetLastError();
}

size_t entropy_ws_bytes(int64_t) { return sizeof(uint32_t) * kCountDirect + sizeof(EntPartial) * kEntGrid; }

hipError_t launch_entropy(const uint32_t *hist, int64_t bins, double *result, void *ws,
                          hipStream_t s) {
    uint32_t *cc = (uint32_t *)ws;
    EntPartial *part = (EntPartial *)(cc + kCountDirect);
    int g = (int)std::min<int64_t>(kEntGrid, std::max<int64_t>(1, cdiv(bins, kBlock)));
    hipLaunchKernelGGL(k_entropy_counts, dim3(g), dim3(kBlock), 0, s, hist, bins, cc, part);
    hipLaunchKernelGGL(k_entropy_final, dim3(1), dim3(kFinalBlock), 0, s, (const uint32_t *)cc,
                       (const EntPartial *)part, g, result);
    return hipGetLastError();
}

int32_t entropy_regions_count(int32_t grid_r, int32_t grid_c, const int32_t *levels,
                              int32_t nlevels) {
    int32_t n = 0;
    for (int32_t i = 0; i < nlevels; ++i)
        n += std::min(levels[i], grid_r) * std::min(levels[i], grid_c);
    return n;
}

size_t entropy_regions_ws_bytes(int32_t grid_r, int32_t grid_c, const int32_t *levels,
                                int32_t nlevels) {
    const int32_t n = entropy_regions_count(grid_r, grid_c, levels, nlevels);
    return sizeof(EntPartial) * (size_t)n * (size_t)region_parts(grid_r, grid_c, levels, nlevels, n);
}

hipError_t launch_entropy_regions(const uint32_t *hist, int32_t grid_r, int32_t grid_c,
                                  const int32_t *levels, int32_t nlevels, double *result,
                                  void *ws, hipStream_t s) {
    Levels l{};
    if (nlevels > (int32_t)(sizeof l.level / sizeof l.level[0])) return hipErrorInvalidValue;
    l.n = nlevels;
    std::copy(levels, levels + nlevels, l.level);
    const int32_t n = entropy_regions_count(grid_r, grid_c, levels, nlevels);
    if (n == 0) return hipSuccess;
    const int32_t parts = region_parts(grid_r, grid_c, levels, nlevels, n);
    EntPartial *part = (EntPartial *)ws;
    hipLaunchKernelGGL(k_entropy_regions, dim3((unsigned)((int64_t)n * parts)), dim3(kRegBlock), 0, s, hist,
                       grid_r, grid_c, l, parts, part, result);
    if (parts > 1)
        hipLaunchKernelGGL(k_entropy_regions_final, dim3((unsigned)n), dim3(kWave), 0, s, (const EntPartial *)part,
                           parts, result);
    return hipGetLastError();
}

}  // namespace mxe
