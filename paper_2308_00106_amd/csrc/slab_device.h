// The column-slab product of one workgroup block, shared by the slab SpMV
// kernel (one block per workgroup) and the persistent batch kernel (blocks of
// many matrices pulled from per-XCD queues). Layout and geometry: SlabGeom in
// internal.h, built by kernels_slab.hip.
#pragma once

#include "device_common.h"
#include "internal.h"

namespace mxe {

constexpr int kSlabBlock = 1024;                    // 16 wavefronts
constexpr int kSubBlocks = kSlabBlock / kWave;      // wavefront sub-blocks per block
constexpr int kSlabMax = 64;                        // column slabs per layout
// 64-entry chunks each wavefront keeps in flight. IF = 0 (the single-product
// kernels): 64 bytes of x per lane, at most four chunks. With several
// right-hand sides a wavefront has about one chunk per slab, so a chunk past
// the group's end is skipped, but two of a group wait for their x together.
// IF > 0 (the persistent batch kernel): as many as keep about IF bytes of x
// per lane in flight, 1 to 8.
template <int KM, typename T, int IF> struct SlabUnroll {
    static constexpr int B = IF / (KM * (int)sizeof(T));
    static constexpr int F = 64 / (KM * (int)sizeof(T)), L = F < 1 ? 1 : F > 4 ? 4 : F;
    static constexpr int value = IF == 0 ? L : B < 1 ? 1 : B > 8 ? 8 : B;
};
template <typename V, typename T> struct SlabVal;
template <> struct SlabVal<double, double> {
    __device__ static double get(double v) { return v; }
};
template <> struct SlabVal<float, float> {
    __device__ static float get(float v) { return v; }
};
template <> struct SlabVal<uint16_t, float> {
    __device__ static float get(uint16_t v) { return bf16_to_f32(v); }
};

// The k values of an X row, 16 bytes at a time as long as they last, whatever
// the row's alignment: 16 bytes of a row cost the L1 one access, as a single
// value does. 500K rows of 12 FP32 entries with 5 right-hand sides take 79 us,
// read value by value 112.
template <typename T, int KM>
__device__ __attribute__((always_inline)) inline void load_x(const char *row, int32_t k, T (&x)[KM]) {
    constexpr int W = (16 / (int)sizeof(T)) < KM ? 16 / (int)sizeof(T) : KM;
    typedef T vec_t __attribute__((ext_vector_type(W), aligned(sizeof(T))));
    typedef T two_t __attribute__((ext_vector_type(2), aligned(sizeof(T))));
    const T *xr = reinterpret_cast<const T *>(row);
    if (k == KM) {                                            // no branch between the loads
#pragma unroll
        for (int q = 0; q < KM; q += W) {
            const vec_t w = *reinterpret_cast<const vec_t *>(xr + q);
#pragma unroll
            for (int r = 0; r < W; ++r) x[q + r] = w[r];
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < KM; q += W) {
        if (q + W <= k) {
            const vec_t w = *reinterpret_cast<const vec_t *>(xr + q);
#pragma unroll
            for (int r = 0; r < W; ++r) x[q + r] = w[r];
            continue;
        }
#pragma unroll
        for (int r = 0; r < W; r += 2) {
            if (q + r + 2 <= k) {
                const two_t w = *reinterpret_cast<const two_t *>(xr + q + r);
                x[q + r] = w[0];
                x[q + r + 1] = w[1];
            } else {
                x[q + r] = q + r < k ? xr[q + r] : T(0);
                x[q + r + 1] = T(0);
            }
        }
    }
}

// Block `block` of the layout, by a workgroup of kSlabBlock threads; tid is
// the thread's index in it. The workgroup walks the slabs in a rotation that
// starts at the slab tied to XCD `xcd` (its own XCD; in a batch, the XCD of
// the queue the block came from), all together (a barrier after each slab),
// so its wavefronts gather from the same L2-resident x slice; inside a slab a
// wavefront loads up to SlabUnroll<KM, T, IF> chunks of its group at once, issues their x
// gathers together, then reduces each chunk by row. The first batch of the
// next slab's group is loaded before each barrier. yp: LDS for the block's
// partial y (rows_per_block x KM values of T); soff: LDS for the wavefronts'
// group offsets; x32: slab_x32, 32-bit offsets of X rows. The
// caller separates two calls on one workgroup by a barrier.
// WIN: X rows [w0, w0 + win) are first copied to LDS (xw, win x KM values of
// T), and entries whose column falls there read x from LDS instead of
// gathering it (the same values, so the same sums).
// ycol (may be null): column q of the result goes to ycol[q] (its row 0)
// with leading dimension ycol_ld[q] instead of Y + q with ldy.
// What bounds it: with one right-hand side the L2's request rate (one per
// entry), with several the latency of a slab's gathers and the wavefronts'
// instructions. With the sums' idle steps left out (segmented_scan), two chunks
// in flight and 24-bit row offsets, 1.16M rows of 12 FP32 entries and k = 8 went
// from 153 to 116 us (0.75 MiB slabs), 700K rows of 10 FP64 entries and k = 4
// from 122 to 63.
// prio (one right-hand side): the wavefront raises its issue priority while
// it sends out a batch's x gathers and drops it for the reductions.
template <typename V, typename T, int KM, int SR, bool WIN = false, int IF = 0>
__device__ __attribute__((always_inline)) inline void
slab_block(const SlabGeom &g, int32_t block, int xcd, const int32_t *__restrict__ off,
           const uint32_t *__restrict__ idx, const V *__restrict__ val, int32_t k,
           const T *__restrict__ X, int64_t ldx, T *__restrict__ Y, int64_t ldy, int x32,
           T *yp, int32_t (*soff)[kSlabMax + 1], int tid, T *xw = nullptr, int32_t w0 = 0,
           int32_t win = 0, void *const *ycol = nullptr, const int64_t *ycol_ld = nullptr,
           bool prio = false) {
    using S = Semiring<SR, T>;
    const int wave = tid / kWave, lane = tid % kWave;
    const int32_t R = g.rows_per_block;
    for (int i = tid; i < R * KM; i += kSlabBlock) yp[i] = S::identity();
    if constexpr (WIN) {
        for (int32_t i = tid; i < win * KM; i += kSlabBlock) {
            const int32_t r = w0 + i / KM, q = i % KM;
            xw[i] = (r < g.ncols && (KM == 1 || q < k)) ? X[(int64_t)r * ldx + q] : T(0);
        }
    }
    T *ywave = yp + (int64_t)wave * g.rows_per_sub * KM;
    // this wavefront's groups (one per slab) and their offsets
    const int32_t *o = off + ((int64_t)block * kSubBlocks + wave) * g.slabs;
    for (int s = lane; s <= g.slabs; s += kWave) soff[wave][s] = o[s];
    __syncthreads();
    const int s0 = (int)(((int64_t)xcd * g.slabs) / 8);
    const uint32_t cmask = (1u << g.cbits) - 1u;
    constexpr int kD = SlabUnroll<KM, T, IF>::value;
    uint32_t u[kD];
    // values as stored, widened where they are used: widening BF16 here, in
    // the branch that loads it, made each chunk wait for its value before the
    // next chunk's loads went out
    V a[kD];
    auto load_batch = [&](int32_t c, int32_t e) {             // up to kD chunks of [c, e)
#pragma unroll
        for (int j = 0; j < kD; ++j) {
            const int32_t p = c + j * kWave + lane;
            const bool v = p < e;
            u[j] = v ? idx[p] : 0xffffffffu;
            a[j] = v ? val[p] : V{};
        }
    };
    load_batch(soff[wave][s0], soff[wave][s0 + 1]);
    for (int t = 0; t < g.slabs; ++t) {                       // same count in every wavefront
        const int s = s0 + t < g.slabs ? s0 + t : s0 + t - g.slabs;
        int32_t b = soff[wave][s], e = soff[wave][s + 1];
        // scalar bounds, but for the single product of one right-hand side: 1.7M
        // FP64 rows of 14 took 147 us with them, 145.5 without, three matrices in
        // turn; the batch of 16 FP32 matrices 392 and 399
        if constexpr (KM > 1 || IF > 0) {
            b = __builtin_amdgcn_readfirstlane(b);
            e = __builtin_amdgcn_readfirstlane(e);
        }
        for (int32_t c = b; c < e; c += kD * kWave) {
            if (c != b) load_batch(c, e);                     // the first batch is already loaded
            T xv[kD][KM];
            if constexpr (KM == 1) {
                if (prio) __builtin_amdgcn_s_setprio(2);
            }
#pragma unroll
            for (int j = 0; j < kD; ++j) {
                if (KM > 2 && j > 0 && c + j * kWave >= e) break;      // uniform per wavefront
                const bool v = u[j] != 0xffffffffu;
                if constexpr (WIN) {
                    const uint32_t d = (u[j] & cmask) - (uint32_t)w0;
                    if (v && d < (uint32_t)win) {
#pragma unroll
                        for (int q = 0; q < KM; ++q) xv[j][q] = xw[(int64_t)d * KM + q];
                        continue;
                    }
                }
                const uint32_t col = v ? u[j] & cmask : 0;        // padding reads row 0 into no row's sum
                if constexpr (KM == 1) {
                    xv[j][0] = v ? X[(int64_t)col * ldx] : T(0);
                } else if (x32) {
                    load_x<T, KM>(reinterpret_cast<const char *>(X) + __umul24(col, (uint32_t)ldx * (uint32_t)sizeof(T)),
                                  k, xv[j]);
                } else {
                    load_x<T, KM>(reinterpret_cast<const char *>(X + (int64_t)col * ldx), k, xv[j]);
                }
            }
            if constexpr (KM == 1) {
                if (prio) __builtin_amdgcn_s_setprio(0);
            }
#pragma unroll
            for (int j = 0; j < kD; ++j) {
                if (c + j * kWave >= e) break;                // uniform per wavefront
                // padding lanes (key 0xffffffff) sit after every valid lane
                const uint32_t key = u[j] != 0xffffffffu ? (u[j] >> g.cbits) : 0xffffffffu;
                const T aj = SlabVal<V, T>::get(a[j]);
                T prod[KM];
#pragma unroll
                for (int q = 0; q < KM; ++q) prod[q] = S::mul(aj, xv[j][q]);
                bool tail;                                    // the last lane of each row
                // every step up to two right-hand sides: their chunks hold rows of
                // several entries, and finding the idle steps costs more than they
                // do (k = 2, 800K skewed FP32 rows in their own order 41.7 us, so
                // 38.9; 700K permuted rows of 8 38.5 and 37.3); not in the batch,
                // where small groups leave more steps idle (391 us, so 396)
                if constexpr (KM == 1 || (KM == 2 && IF == 0)) {
                    if constexpr (SR == 0) segmented_scan<true>(key, 0, prod);
                    else segmented_scan_op<true, S>(key, 0, prod);
                    const uint32_t nxt = __shfl_down(key, 1);
                    tail = key != 0xffffffffu && (lane == kWave - 1 || nxt != key);
                } else {
                    const uint64_t same = same_as_before(key);
                    if constexpr (SR == 0) segmented_scan<false>(key, same, prod);
                    else segmented_scan_op<false, S>(key, same, prod);
                    tail = in_lanes(__builtin_amdgcn_ballot_w64(key != 0xffffffffu) & ~(same >> 1));
                }
                if (tail) {
#pragma unroll
                    for (int q = 0; q < KM; ++q)
                        ywave[(int64_t)key * KM + q] = S::add(ywave[(int64_t)key * KM + q], prod[q]);
                }
                // the next chunk's tails may update the same rows: keep order
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
        if (t + 1 < g.slabs) {                                // next slab's first batch, issued
            const int sn = s + 1 < g.slabs ? s + 1 : 0;       // before the barrier waits
            load_batch(soff[wave][sn], soff[wave][sn + 1]);
        }
        __syncthreads();
    }
    const int64_t row0 = (int64_t)block * R;
    for (int i = tid; i < R * KM; i += kSlabBlock) {
        const int64_t row = row0 + i / KM;
        const int q = i % KM;
        if (row < g.nrows && (KM == 1 || q < k)) {
            // y is streamed out: non-temporal stores leave no dirty lines in
            // the L2 for the end of the launch to write back
            if (ycol) __builtin_nontemporal_store(yp[i], &as_global(static_cast<T *>(ycol[q]))[row * ycol_ld[q]]);
            else __builtin_nontemporal_store(yp[i], &Y[row * ldy + q]);
        }
    }
}

}  // namespace mxe
