// Column-panel SpMV for gfx950, one right-hand side: the x gathers of a
// max-entropy matrix made from LDS, in two streaming passes.
//
// The column-slab kernel (kernels_slab.hip) gathers each x from the XCD's L2
// and is bound by the L2's request rate, about one request per entry: 48.7M
// FP32 entries over 4M columns take 288 us, whatever the value type. Here no x
// is gathered from memory at all. Columns are cut into panels whose x fills
// 64 KiB of LDS, rows into chunks whose products fill 128 KiB of LDS:
//
//   1. k_panel_products: a workgroup copies one panel's x into LDS, streams a
//      share of the panel's entries (value and a 16-bit offset of its x) and
//      streams their products out, in the same order;
//   2. k_panel_rows: a workgroup per CU walks chunks: it collects a chunk's
//      products, one run of consecutive entries per panel, puts each at its row
//      order's place in LDS (a 16-bit index per entry) and sums the rows there.
//
// Both passes move whole cache lines only, 2 sizeof(T) + sizeof(V) + 4 bytes
// per entry, and run at the rate of memory: the FP32 matrix above takes 90 us
// (520 MB, 5.7 TB/s) and 86 us (325 MB, 3.8 TB/s), its BF16 form of 1.5M rows
// 30 + 32 us where the slab kernel takes 106. FP64 entries move 28 bytes, 2M
// rows of 10 take 67 + 45 us, about what the slab kernel's gathers take, so the
// tuner times both. In the first pass two workgroups of 1024 threads fit a CU;
// 128 KiB panels (one per CU) made it 6% slower. In the second one workgroup per
// CU with twice the chunk, so runs twice as long, and the next chunk's products
// on their way while it sums takes 92 / 36 / 60 us (FP32 / BF16 / FP64, new
// matrices in turn) where two with 64 KiB took 97 / 38 / 66; its products alone
// take 64 and summing 20, which two workgroups half a chunk apart hid no better.
// With several right-hand sides the products grow with k while a gather of k
// values stays one request, so those stay with the slab kernel.
//
// Without memory for the products the second pass makes them itself, x gathered
// from memory (launch_spmv_panel): the same products summed the same way, so the
// same bits, but at a gather per entry. The FP32, BF16 and FP64 matrices above
// take 547, 180 and 239 us so, where they take 180, 67 and 118 with the workspace
// and 752, 188 and 317 as row-group products of eight lanes.
//
// Rows are summed in a fixed order (positions in groups, groups in row
// order), so results are deterministic.

#include "device_common.h"
#include "internal.h"

#include <algorithm>
#include <type_traits>

namespace mxe {

namespace {

constexpr int kPanelBlock = 1024;
constexpr int kPanelWaves = kPanelBlock / kWave;
constexpr int kPanelMax = 1024;                    // panels per layout
constexpr int kPanelBytes = 65536;                 // of x in LDS per workgroup
constexpr int kChunkBytes = 131072;                // of products in LDS per workgroup
constexpr int kRowSlice = 4096;                    // row starts of a chunk kept in LDS
constexpr int kPanelMinRun = 8;                    // mean entries of a run, at least

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <typename V, typename T> struct PanelVal;
template <> struct PanelVal<double, double> {
    __device__ static double get(double v) { return v; }
};
template <> struct PanelVal<float, float> {
    __device__ static float get(float v) { return v; }
};
template <> struct PanelVal<uint16_t, float> {
    __device__ static float get(uint16_t v) { return bf16_to_f32(v); }
};

// ---- layout build ---------------------------------------------------------------
// Entries are stored panel by panel, inside a panel chunk by chunk; each
// (panel, chunk) run is padded to a multiple of four entries, so that both
// passes read and write whole groups of four. A padding entry is a zero at
// the panel's first column whose product goes to a place no row has.

// crow[b] = first row whose entries start at or after b * quota
__global__ __launch_bounds__(256) void k_panel_chunks(PanelGeom g, const int32_t *__restrict__ rp,
                                                      int32_t *__restrict__ crow) {
    const int32_t b = blockIdx.x * 256 + threadIdx.x;
    if (b > g.chunks) return;
    if (b == g.chunks) {
        crow[b] = g.nrows;
        return;
    }
    const int64_t lim = (int64_t)b * g.quota;
    int32_t lo = 0, hi = g.nrows;                   // first row with rp[row] >= lim
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (rp[mid] < lim) lo = mid + 1;
        else hi = mid;
    }
    crow[b] = lo;
}

// Pass 1 of the build: cnt[p * chunks + b] = entries of chunk b in panel p,
// rounded up to four
__global__ __launch_bounds__(kPanelBlock) void k_panel_count(PanelGeom g, const int32_t *__restrict__ rp,
                                                             const int32_t *__restrict__ col,
                                                             const int32_t *__restrict__ crow,
                                                             int32_t *__restrict__ cnt) {
    __shared__ int32_t c[kPanelMax];
    const int32_t b = blockIdx.x;
    for (int p = threadIdx.x; p < g.panels; p += kPanelBlock) c[p] = 0;
    __syncthreads();
    const int32_t e0 = rp[crow[b]], e1 = rp[crow[b + 1]];
    for (int32_t e = e0 + threadIdx.x; e < e1; e += 4 * kPanelBlock) {
        int32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = e + j * kPanelBlock < e1 ? col[e + j * kPanelBlock] : -1;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (v[j] >= 0) atomicAdd(&c[v[j] >> g.wbits], 1);
    }
    __syncthreads();
    for (int p = threadIdx.x; p < g.panels; p += kPanelBlock) cnt[(int64_t)p * g.chunks + b] = (c[p] + 3) & ~3;
}

// place in LDS of position i of a chunk: a thread's positions lie a workgroup's
// width apart
template <int EB>
__device__ inline uint32_t place(uint32_t i) {
    constexpr uint32_t E = kChunkBytes / EB / kPanelBlock;
    return (i % E) * kPanelBlock + i / E;
}

// Pass 2 of the build: a workgroup orders its chunk's entries by panel in LDS
// (an LDS cursor per panel; the order inside a run does not matter, every
// entry carries its place in the chunk), then writes the runs out four
// entries per lane.
template <typename V, int EB>
__global__ __launch_bounds__(kPanelBlock) void k_panel_fill(
    PanelGeom g, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const V *__restrict__ val, const int32_t *__restrict__ crow, const int32_t *__restrict__ off,
    int32_t *__restrict__ offt, uint16_t *__restrict__ c16, uint16_t *__restrict__ pos16,
    V *__restrict__ val_out) {
    extern __shared__ uint32_t srt[];               // entries by panel: column << 16 | position
    __shared__ int32_t gbeg[kPanelMax], lbeg[kPanelMax + 1], cur[kPanelMax];
    __shared__ int32_t wsum[kPanelWaves];
    const int32_t b = blockIdx.x, t = threadIdx.x;
    int32_t len = 0;
    if (t < g.panels) {
        const int64_t o = (int64_t)t * g.chunks + b;
        const int32_t s = off[o], e = off[o + 1];
        gbeg[t] = s;
        len = e - s;
        offt[(int64_t)b * g.panels + t] = s;
        if (b == g.chunks - 1) offt[(int64_t)g.chunks * g.panels + t] = e;
    }
    int32_t inc = len;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t v = __shfl_up(inc, o);
        if (t % kWave >= o) inc += v;
    }
    if (t % kWave == kWave - 1) wsum[t / kWave] = inc;
    __syncthreads();
    int32_t base = 0;
    for (int w = 0; w < t / kWave; ++w) base += wsum[w];
    if (t < g.panels) {
        lbeg[t] = cur[t] = base + inc - len;
        if (t == g.panels - 1) lbeg[g.panels] = base + inc;
    }
    __syncthreads();
    // padding entries: column 0 of the panel, the spare position past the chunk
    const int32_t padded = lbeg[g.panels];
    for (int32_t i = t; i < padded; i += kPanelBlock) srt[i] = (uint32_t)g.cap;
    __syncthreads();
    const int32_t e0 = rp[crow[b]], n = rp[crow[b + 1]] - e0;
    const uint32_t cmask = (1u << g.wbits) - 1u;
    for (int32_t i = t; i < n; i += 4 * kPanelBlock) {
        int32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = i + j * kPanelBlock < n ? col[e0 + i + j * kPanelBlock] : -1;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (v[j] >= 0) {
                const int32_t s = atomicAdd(&cur[v[j] >> g.wbits], 1);
                srt[s] = ((uint32_t)v[j] & cmask) << 16 | (uint32_t)(i + j * kPanelBlock);
            }
    }
    __syncthreads();
    constexpr int G = 16;
    typedef V vv __attribute__((ext_vector_type(4)));
    typedef uint16_t hv __attribute__((ext_vector_type(4)));
    for (int p = t / G; p < g.panels; p += kPanelBlock / G) {
        const int32_t s = lbeg[p], cntp = lbeg[p + 1] - s, o = gbeg[p];
        for (int32_t i = 4 * (t % G); i < cntp; i += 4 * G) {
            vv v;
            hv c, q;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t w = srt[s + i + j], at = w & 0xffffu;
                v[j] = at == (uint32_t)g.cap ? V(0) : val[e0 + at];
                c[j] = (uint16_t)((w >> 16) * EB);
                q[j] = (uint16_t)place<EB>(at);
            }
            *reinterpret_cast<vv *>(val_out + o + i) = v;
            *reinterpret_cast<hv *>(c16 + o + i) = c;
            *reinterpret_cast<hv *>(pos16 + o + i) = q;
        }
    }
}

// ---- the product -------------------------------------------------------------------

// Entries per lane and load: 16 bytes of value where that is at most 4 entries.
template <typename V> struct PanelVec { static constexpr int N = sizeof(V) == 8 ? 2 : 4; };  // divides the runs' 4

template <int SR, typename V, typename T>
__device__ inline T panel_product(V v, T x) {
    return Semiring<SR, T>::mul(PanelVal<V, T>::get(v), x);
}

// First pass. Bound by memory bandwidth: value and offset read and product
// written once, x copied to LDS by each of the panel's `split` workgroups
// (blockIdx / split is the panel). The entries' loads run two groups ahead of
// their use and the first go out before the copy of x.
template <typename V, typename T, int SR>
__global__ __launch_bounds__(kPanelBlock) void k_panel_products(
    PanelGeom g, const int32_t *__restrict__ offt, const uint16_t *__restrict__ c16,
    const V *__restrict__ val, const T *__restrict__ X, int64_t ldx, T *__restrict__ prod) {
    __shared__ T xs[kPanelBytes / sizeof(T)];
    constexpr int N = PanelVec<V>::N, U = 2;
    typedef V vv __attribute__((ext_vector_type(N)));
    typedef uint16_t cv __attribute__((ext_vector_type(N)));
    typedef T tv __attribute__((ext_vector_type(N)));
    const int32_t p = blockIdx.x / g.split, part = blockIdx.x % g.split;
    const int64_t b0 = offt[p], b1 = offt[(int64_t)g.chunks * g.panels + p];
    const int64_t s0 = part == 0 ? b0 : (b0 + (b1 - b0) * part / g.split) & ~3ll;
    const int64_t s1 = part == g.split - 1 ? b1 : (b0 + (b1 - b0) * (part + 1) / g.split) & ~3ll;
    const int64_t q1 = s1 / N;                      // runs, so panels too, are whole groups of 4
    int64_t q = s0 / N + threadIdx.x;
    const vv *va = reinterpret_cast<const vv *>(val);
    const cv *ca = reinterpret_cast<const cv *>(c16);
    vv a[U];
    cv c[U];
    auto load = [&](int64_t at) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = at + u * kPanelBlock;
            if (k < q1) {
                a[u] = __builtin_nontemporal_load(&va[k]);
                c[u] = __builtin_nontemporal_load(&ca[k]);
            }
        }
    };
    load(q);
    const int64_t c0 = (int64_t)p << g.wbits;
    const int32_t w = (int32_t)std::min<int64_t>(int64_t(1) << g.wbits, g.ncols - c0);
    const T *xp = X + c0 * ldx;
    for (int32_t i = threadIdx.x; i < w; i += 8 * kPanelBlock) {
        T x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int32_t k = i + j * kPanelBlock;
            x[j] = k < w ? xp[(int64_t)k * ldx] : T(0);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int32_t k = i + j * kPanelBlock;
            if (k < w) xs[k] = x[j];
        }
    }
    __syncthreads();
    for (; q < q1; q += U * kPanelBlock) {
        tv r[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (q + u * kPanelBlock < q1) {
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    const T x = *reinterpret_cast<const T *>(reinterpret_cast<const char *>(xs) + c[u][n]);
                    r[u][n] = panel_product<SR, V>(V(a[u][n]), x);
                }
            }
        const int64_t at = q;
        load(q + U * kPanelBlock);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = at + u * kPanelBlock;
            if (k < q1) reinterpret_cast<tv *>(prod)[k] = r[u];
        }
    }
}

// LDS written before is visible to the workgroup after it; loads from memory
// stay in flight across it (__syncthreads would wait for them).
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Where the second pass takes four consecutive products of panel p from: the
// first pass's workspace, or the entries and x. Quads by 32-bit byte offsets from
// uniform bases (panel_geometry bounds them).
template <typename T> struct StoredProducts {
    static constexpr int kAhead = sizeof(T) == 8 ? 3 : 5;  // groups of fours of a run in flight per lane
    typedef T tv __attribute__((ext_vector_type(4)));
    const T *prod;
    __device__ tv quad(int32_t a, int) const {
        return *reinterpret_cast<const tv *>(reinterpret_cast<const char *>(prod) + (uint32_t)a * (uint32_t)sizeof(tv));
    }
};
template <typename V, typename T, int SR> struct OwnProducts {
    static constexpr int kAhead = 1;                       // no registers left for more, no memory to spill to
    typedef T tv __attribute__((ext_vector_type(4)));
    typedef V vv __attribute__((ext_vector_type(4)));
    typedef uint16_t cv __attribute__((ext_vector_type(4)));
    const V *val;
    const uint16_t *c16;
    const T *X;
    int64_t ldx;
    int32_t wbits;
    __device__ tv quad(int32_t a, int p) const {
        const vv v = reinterpret_cast<const vv *>(val)[a];
        const cv c = reinterpret_cast<const cv *>(c16)[a];
        const T *xp = X + ((int64_t)p << wbits) * ldx;
        tv r;
#pragma unroll
        for (int n = 0; n < 4; ++n)
            r[n] = panel_product<SR, V>(V(v[n]), xp[(int64_t)(c[n] / sizeof(T)) * ldx]);
        return r;
    }
};

// Second pass: a workgroup per CU walks its chunks, the next chunk's products
// on their way to registers while it sums the current one. G lanes share a run,
// each lane taking four entries at a time; R runs of up to U groups of G fours
// are in flight per lane, what lies past them is read when the chunk's turn
// comes. A chunk's place i lies at (i % E, i / E) of an E x 1024 array, so
// that thread t sums places [E t, E t + E) by row without bank conflicts (a
// bit per place marks the row starts); a row's sum is then the last partial
// sum of each group of E it spans. Summing with one to eight lanes per row
// over its places instead took 13% longer (rows of 1 to 256 entries: the longest
// row of a wavefront held up the others).
template <typename Src, typename T, int SR, int G, int R, int U>
__global__ __launch_bounds__(kPanelBlock) void k_panel_rows(
    PanelGeom g, const int32_t *__restrict__ offt, const int32_t *__restrict__ crow,
    const int32_t *__restrict__ rp, const uint16_t *__restrict__ pos16, Src products,
    T *__restrict__ Y, int64_t ldy) {
    constexpr int E = kChunkBytes / (int)sizeof(T) / kPanelBlock;     // positions per thread
    constexpr int RP = 3;                                             // row starts per thread held ahead
    __shared__ T sp[E * kPanelBlock];
    __shared__ int32_t rs[kRowSlice + 1];
    __shared__ uint32_t mask[E * kPanelBlock / 32 + 1];
    // FP32 products are summed in FP64: a row's terms stand in a line here, where
    // the other products' lanes add them as a tree
    using A = std::conditional_t<SR == 0, double, T>;
    using Sum = Semiring<SR, A>;
    constexpr int NG = kPanelBlock / G;
    typedef T tv __attribute__((ext_vector_type(4)));
    typedef uint16_t pv __attribute__((ext_vector_type(4)));
    // neighbouring chunks share cache lines at the ends of their runs: each
    // XCD takes a contiguous range of chunks, its workgroups side by side in it
    const int32_t per = (g.chunks + 7) / 8, side = (int32_t)gridDim.x / 8;
    const int32_t c0 = (int32_t)(blockIdx.x % 8) * per, c1 = min(c0 + per, g.chunks);
    int32_t b = c0 + (int32_t)(blockIdx.x / 8);
    if (b >= c1) return;
    auto posv = [&](int32_t a) {
        return *reinterpret_cast<const pv *>(reinterpret_cast<const char *>(pos16) + (uint32_t)a * (uint32_t)sizeof(pv));
    };
    auto put = [&](tv a, pv q) {
#pragma unroll
        for (int n = 0; n < 4; ++n) sp[q[n]] = a[n];
    };
    const int t = threadIdx.x, lane = t % G;
    int32_t a[R], n[R];                             // first quad and end of the chunk's runs t / G + r NG
    int32_t a1[R], n1[R], r1 = 0, rows1 = 0;        // the same of the chunk after it
    int32_t start[RP], r0 = 0, rows = 0, e0 = 0;
    tv v[R][U];
    pv w[R][U];
    auto offsets = [&](int32_t c) {
        const int32_t *o0 = offt + (int64_t)c * g.panels, *o1 = o0 + g.panels;
        r1 = crow[c];
        rows1 = crow[c + 1] - r1;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int32_t p = min(t / G + r * NG, g.panels - 1);
            a1[r] = (o0[p] >> 2) + lane;
            n1[r] = t / G + r * NG < g.panels ? o1[p] >> 2 : 0;
        }
    };
    auto fetch = [&]() {                            // the chunk whose offsets have come
        r0 = r1;
        rows = rows1;
        e0 = rp[r0];
#pragma unroll
        for (int k = 0; k < RP; ++k) start[k] = rp[r0 + min(t + k * kPanelBlock, rows)];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            a[r] = a1[r];
            n[r] = n1[r];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (a[r] + u * G < n[r]) {
                    v[r][u] = products.quad(a[r] + u * G, t / G + r * NG);
                    w[r][u] = posv(a[r] + u * G);
                }
        }
    };
    offsets(b);
    fetch();
    for (;;) {
        if (b + side < c1) offsets(b + side);
        for (int i = t; i <= E * kPanelBlock / 32; i += kPanelBlock) mask[i] = 0;
        lds_barrier();                              // the previous chunk's sums have been read as well
        auto mark = [&](int i, int32_t s) {
            if (i <= kRowSlice) rs[i] = s;
            atomicOr(&mask[s >> 5], 1u << (s & 31));
        };
#pragma unroll
        for (int k = 0; k < RP; ++k)
            if (t + k * kPanelBlock <= rows) mark(t + k * kPanelBlock, start[k] - e0);
        for (int i = t + RP * kPanelBlock; i <= rows; i += kPanelBlock) mark(i, rp[r0 + i] - e0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (a[r] + u * G < n[r]) put(v[r][u], w[r][u]);
            for (int32_t q = a[r] + U * G; q < n[r]; q += G) put(products.quad(q, t / G + r * NG), posv(q));
        }
        for (int p = t / G + R * NG; p < g.panels; p += NG) {
            const int32_t o = offt[(int64_t)b * g.panels + p] >> 2, e = offt[(int64_t)(b + 1) * g.panels + p] >> 2;
            for (int32_t q = o + lane; q < e; q += G) put(products.quad(q, p), posv(q));
        }
        const int32_t row0 = r0, nrow = rows, first = e0;
        b += side;
        if (b < c1) fetch();
        lds_barrier();
        // positions [E t, E t + E): running sums by row
        {
            const uint32_t m = mask[t * E >> 5] >> (t * E & 31);
            A acc = sp[t];
#pragma unroll
            for (int j = 1; j < E; ++j) {
                const A x = sp[j * kPanelBlock + t];
                acc = (m >> j & 1) ? x : Sum::add(acc, x);
                sp[j * kPanelBlock + t] = (T)acc;
            }
        }
        lds_barrier();
        for (int32_t i = t; i < nrow; i += kPanelBlock) {
            const int32_t s = i < kRowSlice ? rs[i] : rp[row0 + i] - first;
            const int32_t last = (i < kRowSlice ? rs[i + 1] : rp[row0 + i + 1] - first) - 1;
            A acc = Sum::identity();
            for (int32_t q = s / E; q <= last / E && s <= last; ++q) {
                const int32_t j = min(last, q * E + E - 1) % E;
                acc = Sum::add(acc, A(sp[j * kPanelBlock + q]));
            }
            __builtin_nontemporal_store((T)acc, &Y[(int64_t)(row0 + i) * ldy]);
        }
        if (b >= c1) break;
    }
}

template <typename T, int SR, typename Src>
void rows_launch(const PanelGeom &g, const PanelLayout &l, const int32_t *rp, const Src &products, void *Y,
                 int64_t ldy, hipStream_t s) {
    const int32_t per = (g.chunks + 7) / 8, side = std::max(1, std::min(per, g.cus / 8));
    hipLaunchKernelGGL((k_panel_rows<Src, T, SR, 8, 2, Src::kAhead>), dim3(8 * side), dim3(kPanelBlock), 0,
                       s, g, l.offt, l.crow, rp, l.pos16, products, (T *)Y, ldy);
}

template <typename V, typename T, int SR>
hipError_t panel_launch(const PanelGeom &g, const PanelLayout &l, const int32_t *rp, const void *X,
                        int64_t ldx, void *Y, int64_t ldy, void *prod, hipStream_t s) {
    if (prod) {
        hipLaunchKernelGGL((k_panel_products<V, T, SR>), dim3(g.panels * g.split), dim3(kPanelBlock), 0, s,
                           g, l.offt, l.c16, (const V *)l.val, (const T *)X, ldx, (T *)prod);
        rows_launch<T, SR>(g, l, rp, StoredProducts<T>{(const T *)prod}, Y, ldy, s);
    } else {
        const OwnProducts<V, T, SR> own{(const V *)l.val, l.c16, (const T *)X, ldx, g.wbits};
        rows_launch<T, SR>(g, l, rp, own, Y, ldy, s);
    }
    return hipGetLastError();
}

template <typename V, typename T>
hipError_t panel_by_semiring(const PanelGeom &g, const PanelLayout &l, int semiring, const int32_t *rp,
                             const void *X, int64_t ldx, void *Y, int64_t ldy, void *prod,
                             hipStream_t s) {
    switch (semiring) {
    case 0: return panel_launch<V, T, 0>(g, l, rp, X, ldx, Y, ldy, prod, s);
    case 1: return panel_launch<V, T, 1>(g, l, rp, X, ldx, Y, ldy, prod, s);
    case 2: return panel_launch<V, T, 2>(g, l, rp, X, ldx, Y, ldy, prod, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool panel_geometry(int32_t nrows, int32_t ncols, int64_t nnz, int32_t max_row, int vtype, int cu_count,
                    PanelGeom *g) {
    if (nrows <= 0 || ncols <= 0 || nnz <= 0 || max_row < 1) return false;
    const int eb = vtype == VAL_F64 ? 8 : 4;
    int wbits = 0;
    while ((eb << (wbits + 1)) <= kPanelBytes) ++wbits;
    const int64_t panels = cdiv(ncols, int64_t(1) << wbits);
    const int32_t cap = kChunkBytes / eb - 1;       // one place is left for the padding entries
    if (panels > kPanelMax || max_row > cap / 2) return false;
    const int64_t slots = 2 * (int64_t)cu_count;    // workgroups resident at once in the first pass
    // a chunk starts its rows within `quota` entries and ends its last one at
    // most max_row later; as many chunks as fill whole waves of workgroups,
    // with at least an entry per thread
    const int64_t most = cap - max_row;
    const int64_t waves = cdiv(nnz, most * cu_count);
    const int64_t quota = std::min<int64_t>(most, std::max<int64_t>(kPanelBlock, cdiv(nnz, waves * cu_count)));
    // runs of a few entries would be mostly padding
    if (quota < kPanelMinRun * panels) return false;
    g->nrows = nrows;
    g->ncols = ncols;
    g->nnz = nnz;
    g->wbits = wbits;
    g->panels = (int32_t)panels;
    g->cap = cap;
    g->cus = cu_count;
    g->quota = (int32_t)quota;
    g->chunks = (int32_t)cdiv(nnz, quota);
    // workgroups per panel: fill the chip, with at least 4096 entries each
    g->split = (int32_t)std::max<int64_t>(1, std::min<int64_t>(slots / panels, nnz / panels / 4096));
    // 32-bit byte offsets of the products and positions
    return (int64_t)panel_entries(*g) * eb < (int64_t(1) << 32) &&
           (int64_t)panel_entries(*g) < INT32_MAX && panels * g->chunks < INT32_MAX / 2;
}

size_t panel_offsets_count(const PanelGeom &g) { return ((size_t)g.chunks + 1) * g.panels; }

// every run padded to a multiple of 4
size_t panel_entries(const PanelGeom &g) {
    return (size_t)g.nnz + 3 * (size_t)std::min<int64_t>(g.nnz, (int64_t)g.panels * g.chunks);
}

size_t panel_build_ws_bytes(const PanelGeom &g) {
    const size_t n = (size_t)g.chunks * g.panels + 1;
    return (sizeof(int32_t) * n + 255) / 256 * 256 + scan_ws_bytes((int64_t)n);
}

hipError_t launch_panel_build(const PanelGeom &g, const int32_t *rp, const int32_t *col, const void *val,
                              int val_bytes, const PanelLayout &l, void *ws, hipStream_t s) {
    const int64_t n = (int64_t)g.chunks * g.panels + 1;
    int32_t *off = (int32_t *)ws;
    void *scan_ws = (char *)ws + (sizeof(int32_t) * (size_t)n + 255) / 256 * 256;
    hipLaunchKernelGGL(k_panel_chunks, dim3((unsigned)cdiv(g.chunks + 1, 256)), dim3(256), 0, s, g, rp, l.crow);
    hipError_t e;
    hipLaunchKernelGGL(k_panel_count, dim3(g.chunks), dim3(kPanelBlock), 0, s, g, rp, col,
                       (const int32_t *)l.crow, off);
    if ((e = launch_exclusive_scan(off, off, n, scan_ws, s)) != hipSuccess) return e;
    const size_t lds = sizeof(uint32_t) * ((size_t)g.cap + 3 * (size_t)g.panels);
#define MXE_PANEL_FILL(V, EB)                                                                       \
    hipLaunchKernelGGL((k_panel_fill<V, EB>), dim3(g.chunks), dim3(kPanelBlock), lds, s, g, rp, col,      \
                       (const V *)val, (const int32_t *)l.crow, (const int32_t *)off, l.offt, l.c16, \
                       l.pos16, (V *)l.val)
    switch (val_bytes) {
    case 8: MXE_PANEL_FILL(uint64_t, 8); break;
    case 4: MXE_PANEL_FILL(uint32_t, 4); break;
    case 2: MXE_PANEL_FILL(uint16_t, 4); break;
    default: return hipErrorInvalidValue;
    }
#undef MXE_PANEL_FILL
    return hipGetLastError();
}

hipError_t launch_spmv_panel(const PanelGeom &g, const PanelLayout &l, int vtype, int semiring,
                             const int32_t *rp, const void *X, int64_t ldx, void *Y, int64_t ldy,
                             void *prod, hipStream_t s) {
    switch (vtype) {
    case VAL_F64: return panel_by_semiring<double, double>(g, l, semiring, rp, X, ldx, Y, ldy, prod, s);
    case VAL_F32: return panel_by_semiring<float, float>(g, l, semiring, rp, X, ldx, Y, ldy, prod, s);
    case VAL_BF16: return panel_by_semiring<uint16_t, float>(g, l, semiring, rp, X, ldx, Y, ldy, prod, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mxe
