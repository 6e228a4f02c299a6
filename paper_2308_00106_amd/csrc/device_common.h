// Device helpers shared by the mxe kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mxe {

constexpr int kWave = 64;

// A pointer the caller knows to address device memory, in a form the compiler
// can prove it of. Pointers read from memory (a batch's descriptors) are
// otherwise generic, and accesses through them compile to flat instructions,
// which also count against the LDS wait counter: every LDS wait then waits
// for all loads in flight as well.
template <typename T>
__device__ __attribute__((always_inline)) inline T *as_global(T *p) {
    return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

// ---------------------------------------------------------------------------
// Random keys. The permutation of n items is the stable ascending order of
// key(s, i), the i-th output (i = 0, 1, ...) of SplitMix64 started at state s
// (Steele, Lea and Flood, OOPSLA 2014). SplitMix64 advances its state by the
// golden-ratio increment before each output, so output i is the finaliser
// applied to s + (i + 1) * increment: a counter-based hash, computed per index
// with no state and no memory traffic.
// ---------------------------------------------------------------------------
__host__ __device__ inline uint64_t sm64_key(uint64_t s, uint64_t i) {
    uint64_t z = s + (i + 1ull) * 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// ---------------------------------------------------------------------------
// Exact block index floor(j * g / n) for 0 <= j < n < 2^31, 1 <= g <= 2^20
// (the product stays below 2^51, exact in FP64). The FP64 quotient is within
// one of the true floor; one integer correction step makes it exact.
// ---------------------------------------------------------------------------
__device__ inline int32_t block_index(int64_t j, int64_t g, int64_t n, double inv_n) {
    int64_t num = j * g;
    int64_t q = (int64_t)((double)num * inv_n);
    if (q * n > num) --q;
    else if ((q + 1) * n <= num) ++q;
    return (int32_t)q;
}

// ---------------------------------------------------------------------------
// Double-double arithmetic (about 106 significant bits), built from the
// error-free transformations of Knuth (two-sum) and the exact FMA product.
// Used to evaluate the entropy accurately enough to certify its rounding.
// ---------------------------------------------------------------------------
struct dd { double hi, lo; };

#pragma clang fp contract(off)
__device__ inline dd two_sum(double a, double b) {
    double s = a + b;
    double bb = s - a;
    double e = (a - (s - bb)) + (b - bb);
    return {s, e};
}
__device__ inline dd quick_two_sum(double a, double b) {   // |a| >= |b|
    double s = a + b;
    double e = b - (s - a);
    return {s, e};
}
__device__ inline dd two_prod(double a, double b) {
    double p = a * b;
    double e = __builtin_fma(a, b, -p);
    return {p, e};
}
__device__ inline dd dd_add(dd a, dd b) {
    dd s = two_sum(a.hi, b.hi);
    dd t = two_sum(a.lo, b.lo);
    s.lo += t.hi;
    s = quick_two_sum(s.hi, s.lo);
    s.lo += t.lo;
    return quick_two_sum(s.hi, s.lo);
}
__device__ inline dd dd_neg(dd a) { return {-a.hi, -a.lo}; }
__device__ inline dd dd_sub(dd a, dd b) { return dd_add(a, dd_neg(b)); }
__device__ inline dd dd_mul(dd a, dd b) {
    dd p = two_prod(a.hi, b.hi);
    p.lo += a.hi * b.lo;
    p.lo += a.lo * b.hi;
    return quick_two_sum(p.hi, p.lo);
}
__device__ inline dd dd_mul_d(dd a, double b) {
    dd p = two_prod(a.hi, b);
    p.lo += a.lo * b;
    return quick_two_sum(p.hi, p.lo);
}
__device__ inline dd dd_div(dd a, dd b) {
    // long division: two quotient digits and a correction
    double q1 = a.hi / b.hi;
    dd r = dd_sub(a, dd_mul_d(b, q1));
    double q2 = r.hi / b.hi;
    r = dd_sub(r, dd_mul_d(b, q2));
    double q3 = r.hi / b.hi;
    dd q = quick_two_sum(q1, q2);
    return dd_add(q, dd{q3, 0.0});
}
#pragma clang fp contract(on)

// ln 2 as the nearest double-double (the nearest double, then the nearest
// double to the rest).
__device__ constexpr dd kLn2 = {0x1.62e42fefa39efp-1, 0x1.abc9e3b39803fp-56};

// ln(m) for m in [sqrt(1/2), sqrt(2)]: 2 atanh(u), u = (m - 1) / (m + 1),
// |u| <= 0.1716, summed as u * sum_k u^(2k) / (2k + 1) for k < 24; u^2 < 2^-5.08,
// so the truncated tail is below 2^-120 of the sum. The coefficients, also
// nearest double-doubles, stand in the unrolled code: a chain of 23 steps that
// reads each from memory takes twice as long.
__device__ inline dd dd_ln_reduced(dd m) {
    constexpr int kTerms = 24;
    constexpr dd coef[kTerms] = {
        {0x1.0000000000000p+0, 0x0.0p+0},
        {0x1.5555555555555p-2, 0x1.5555555555555p-56},
        {0x1.999999999999ap-3, -0x1.999999999999ap-57},
        {0x1.2492492492492p-3, 0x1.2492492492492p-57},
        {0x1.c71c71c71c71cp-4, 0x1.c71c71c71c71cp-58},
        {0x1.745d1745d1746p-4, -0x1.745d1745d1746p-59},
        {0x1.3b13b13b13b14p-4, -0x1.3b13b13b13b14p-58},
        {0x1.1111111111111p-4, 0x1.1111111111111p-60},
        {0x1.e1e1e1e1e1e1ep-5, 0x1.e1e1e1e1e1e1ep-61},
        {0x1.af286bca1af28p-5, 0x1.af286bca1af28p-59},
        {0x1.8618618618618p-5, 0x1.8618618618618p-59},
        {0x1.642c8590b2164p-5, 0x1.642c8590b2164p-60},
        {0x1.47ae147ae147bp-5, -0x1.eb851eb851eb8p-61},
        {0x1.2f684bda12f68p-5, 0x1.2f684bda12f68p-59},
        {0x1.1a7b9611a7b96p-5, 0x1.1a7b9611a7b96p-61},
        {0x1.0842108421084p-5, 0x1.0842108421084p-60},
        {0x1.f07c1f07c1f08p-6, -0x1.f07c1f07c1f08p-61},
        {0x1.d41d41d41d41dp-6, 0x1.0750750750750p-60},
        {0x1.bacf914c1bad0p-6, -0x1.bacf914c1bad0p-60},
        {0x1.a41a41a41a41ap-6, 0x1.0690690690690p-60},
        {0x1.8f9c18f9c18fap-6, -0x1.f3831f3831f38p-61},
        {0x1.7d05f417d05f4p-6, 0x1.7d05f417d05f4p-62},
        {0x1.6c16c16c16c17p-6, -0x1.f49f49f49f49fp-61},
        {0x1.5c9882b931057p-6, 0x1.310572620ae4cp-61},
    };
    dd num = dd_sub(m, dd{1.0, 0.0});
    dd den = dd_add(m, dd{1.0, 0.0});
    dd u = dd_div(num, den);
    dd w = dd_mul(u, u);
    dd acc = coef[kTerms - 1];
#pragma unroll
    for (int k = kTerms - 2; k >= 0; --k) acc = dd_add(dd_mul(acc, w), coef[k]);
    dd r = dd_mul(u, acc);
    return dd{2.0 * r.hi, 2.0 * r.lo};
}

// ln(x) for an integer-valued double 1 <= x < 2^53: x = m 2^e with m in
// [sqrt(1/2), sqrt(2)), then ln x = e ln2 + ln m.
__device__ inline dd dd_ln_int(double x) {
    int e;
    double m = __builtin_frexp(x, &e);        // x = m 2^e, m in [0.5, 1)
    m *= 2.0;
    e -= 1;                                   // m in [1, 2)
    if (m > 1.4142135623730951) { m *= 0.5; e += 1; }
    dd lm = dd_ln_reduced(dd{m, 0.0});
    return dd_add(dd_mul_d(kLn2, (double)e), lm);
}

// ---------------------------------------------------------------------------
// Value storage conversions, round to nearest, ties to even, from FP64.
// ---------------------------------------------------------------------------
__device__ inline uint16_t bf16_from_f64(double d) {
    uint64_t u = __double_as_longlong(d);
    uint16_t sign = (uint16_t)((u >> 48) & 0x8000u);
    uint64_t a = u & 0x7fffffffffffffffull;
    if (a > 0x7ff0000000000000ull) return sign | 0x7fc0u;          // NaN
    if (a == 0x7ff0000000000000ull) return sign | 0x7f80u;         // infinity
    int e = (int)(a >> 52) - 1023;                                 // unbiased exponent
    if (e < -134) return sign;                                     // below half the least subnormal
    uint64_t m = (a & 0x000fffffffffffffull) | 0x0010000000000000ull;  // value = m 2^(e-52)
    int qexp = e >= -126 ? e - 7 : -133;                           // BF16 spacing at this value
    int shift = qexp - (e - 52);                                   // 45 .. 53
    uint64_t kept = m >> shift;
    uint64_t rem = m & ((1ull << shift) - 1);
    uint64_t half = 1ull << (shift - 1);
    if (rem > half || (rem == half && (kept & 1))) ++kept;
    if (qexp == -133) return sign | (uint16_t)kept;                // subnormal (kept <= 128)
    // normal: kept in [128, 256]; a carry to 256 moves into the exponent
    uint32_t bits = ((uint32_t)(e + 127) << 7) + (uint32_t)(kept - 128);
    if (bits >= 0x7f80u) return sign | 0x7f80u;                    // overflow
    return sign | (uint16_t)bits;
}

__device__ inline float bf16_to_f32(uint16_t b) {
    return __uint_as_float((uint32_t)b << 16);
}

// Semirings of the product (MXE_SR_* in mxe.h: 0 (+, *), 1 (min, +), 2 (or,
// and)), Section 2: identity of the sum, the product of a value and an x, the
// sum. min and or are exact. A term of (min, +) that is NaN is no path: it
// becomes the identity here, where it arises, since a partial minimum that was
// NaN would keep every term joined to it out of the sum.
template <int SR, typename T> struct Semiring;
template <typename T> struct Semiring<0, T> {
    __device__ static T identity() { return T(0); }
    __device__ static T mul(T a, T x) { return a * x; }
    __device__ static T add(T p, T q) { return p + q; }
};
template <typename T> struct Semiring<1, T> {
    __device__ static T identity() { return T(__builtin_inf()); }
    __device__ static T mul(T a, T x) {
        const T m = a + x;
        return m == m ? m : identity();
    }
    __device__ static T add(T p, T q) { return q < p ? q : p; }
};
template <typename T> struct Semiring<2, T> {
    __device__ static T identity() { return T(0); }
    __device__ static T mul(T a, T x) { return (a != T(0) && x != T(0)) ? T(1) : T(0); }
    __device__ static T add(T p, T q) { return (p != T(0) || q != T(0)) ? T(1) : T(0); }
};

// Inclusive segmented scan over a wavefront whose keys never decrease
// (equal keys are adjacent; real keys stay below 0xfffffffe, padding lanes
// carry 0xffffffff after every real one), on DPP lane moves instead of LDS
// permutes: four row_shr steps inside each row of 16 lanes, then row_bcast:15
// into rows 1 and 3 and row_bcast:31 into rows 2 and 3. A lane adds the moved
// value only when it carries its own key; moves from outside a row read value 0
// (adding nothing), and rows a broadcast skips keep a key no row can have.
// A step in which no lane has anything to take is left out: the wavefront's
// chunk of a wide product holds a few entries of a row at most, and with 8
// right-hand sides the six steps were three quarters of the product's
// instructions (see slab_block for what that cost).
//
// same: the lanes that carry the key of the lane before them.
__device__ inline uint64_t same_as_before(uint32_t key) {
    const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp((int)0xfffffffeu, (int)key, 0x138, 0xf, 0xf,
                                                                false);          // wave_shr:1
    return __builtin_amdgcn_ballot_w64(prev == key && key != 0xffffffffu);
}
__device__ inline bool in_lanes(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// the lanes that take from 1, 2, 4 and 8 lanes before them in their row of
// 16, and whether a run of equal keys crosses the rows' edges
struct ScanSteps {
    uint64_t take[4];
    bool rows01_23, rows1_2;
};
__device__ inline ScanSteps scan_steps(uint64_t same) {
    ScanSteps s;
    const uint64_t s2 = same & (same << 1), s4 = s2 & (s2 << 2), s8 = s4 & (s4 << 4);
    s.take[0] = same & 0xfffefffefffefffeull;
    s.take[1] = s2 & 0xfffcfffcfffcfffcull;
    s.take[2] = s4 & 0xfff0fff0fff0fff0ull;
    s.take[3] = s8 & 0xff00ff00ff00ff00ull;
    s.rows01_23 = same & 0x0001000000010000ull;
    s.rows1_2 = same & 0x0000000100000000ull;
    return s;
}
// CTRL: a row shift, row_shr:n (0x110 + n) or row_shl:n (0x100 + n)
template <int CTRL>
__device__ inline uint32_t dpp_shr_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL, int RMASK>
__device__ inline uint32_t dpp_bcast_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)0xfffffffeu, (int)v, CTRL, RMASK, 0xf, false);
}
template <int CTRL>
__device__ inline double dpp_shr(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ inline float dpp_shr(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL, int RMASK>
__device__ inline double dpp_bcast(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, RMASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, RMASK, 0xf, false);
    return __hiloint2double(hi, lo);
}
template <int CTRL, int RMASK>
__device__ inline float dpp_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, RMASK, 0xf, false));
}

// ALL: every lane's key is compared and no step left out.
template <int N, bool ALL, typename T, int KM>
__device__ inline void scan_shr(uint32_t key, uint64_t take, T (&v)[KM]) {
    constexpr int CTRL = 0x110 + N;                           // row_shr:N
    if constexpr (!ALL) {
        if (take == 0) return;
    }
    if constexpr (sizeof(T) == 4) {
        // FP32: each lane zeroes what the lane N places on in its row must
        // not take (the row_shl:N move of the key gives that lane's key), so
        // the move folds into a DPP add: two instructions per value, not
        // three. The same terms are added in the same order.
        bool keep;
        if constexpr (ALL) keep = dpp_shr_u32<0x100 + N>(key) == key;
        else keep = in_lanes(take >> N);
        T w[KM];                                              // all first: a DPP move waits for its source
#pragma unroll
        for (int q = 0; q < KM; ++q) w[q] = keep ? v[q] : T(0);
        if constexpr (KM > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < KM; ++q) v[q] += dpp_shr<CTRL>(w[q]);
    } else {
        bool mine;
        if constexpr (ALL) mine = dpp_shr_u32<CTRL>(key) == key;
        else mine = in_lanes(take);
#pragma unroll
        for (int q = 0; q < KM; ++q) {
            const T m = dpp_shr<CTRL>(v[q]);
            v[q] += mine ? m : T(0);
        }
    }
}
template <int CTRL, int RMASK, typename T, int KM>
__device__ inline void scan_bcast(uint32_t key, T (&v)[KM]) {
    const bool take = dpp_bcast_u32<CTRL, RMASK>(key) == key;
#pragma unroll
    for (int q = 0; q < KM; ++q) {
        const T m = dpp_bcast<CTRL, RMASK>(v[q]);
        v[q] += take ? m : T(0);
    }
}
// The same scan for an operator other than +: every move, inside a row too,
// reads the operator's identity and the never-matching key where its source
// lane lies outside the row (for min, a moved-in 0 would be wrong).
template <int CTRL, int RMASK, typename Op, typename T, int KM>
__device__ inline void scan_step_op(uint32_t key, T (&v)[KM]) {
    const bool take = (uint32_t)__builtin_amdgcn_update_dpp((int)0xfffffffeu, (int)key, CTRL, RMASK,
                                                            0xf, false) == key;
#pragma unroll
    for (int q = 0; q < KM; ++q) {
        T m;
        if constexpr (sizeof(T) == 8) {
            const double id = Op::identity();
            const int lo = __builtin_amdgcn_update_dpp(__double2loint(id), __double2loint(v[q]), CTRL,
                                                       RMASK, 0xf, false);
            const int hi = __builtin_amdgcn_update_dpp(__double2hiint(id), __double2hiint(v[q]), CTRL,
                                                       RMASK, 0xf, false);
            m = __hiloint2double(hi, lo);
        } else {
            m = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int((float)Op::identity()),
                                                           __float_as_int(v[q]), CTRL, RMASK, 0xf,
                                                           false));
        }
        v[q] = take ? Op::add(v[q], m) : v[q];
    }
}
template <bool ALL, typename Op, typename T, int KM>
__device__ inline void segmented_scan_op(uint32_t key, uint64_t same, T (&v)[KM]) {
    ScanSteps s{};
    if constexpr (!ALL) {
        if (same == 0) return;
        s = scan_steps(same);
    }
    if (ALL || s.take[0]) scan_step_op<0x111, 0xf, Op>(key, v);
    if (ALL || s.take[1]) scan_step_op<0x112, 0xf, Op>(key, v);
    if (ALL || s.take[2]) scan_step_op<0x114, 0xf, Op>(key, v);
    if (ALL || s.take[3]) scan_step_op<0x118, 0xf, Op>(key, v);
    if (ALL || s.rows01_23) scan_step_op<0x142, 0xa, Op>(key, v);
    if (ALL || s.rows1_2) scan_step_op<0x143, 0xc, Op>(key, v);
}

// ALL: the steps in one stream of instructions, for one right-hand side, where
// choosing them costs more than the moves (same is not used then).
template <bool ALL, typename T, int KM>
__device__ inline void segmented_scan(uint32_t key, uint64_t same, T (&v)[KM]) {
    ScanSteps s{};
    if constexpr (!ALL) {
        if (same == 0) return;
        s = scan_steps(same);
    }
    scan_shr<1, ALL>(key, s.take[0], v);
    scan_shr<2, ALL>(key, s.take[1], v);
    scan_shr<4, ALL>(key, s.take[2], v);
    scan_shr<8, ALL>(key, s.take[3], v);
    if (ALL || s.rows01_23) scan_bcast<0x142, 0xa>(key, v);   // row_bcast:15 -> rows 1, 3
    if (ALL || s.rows1_2) scan_bcast<0x143, 0xc>(key, v);     // row_bcast:31 -> rows 2, 3
}

}  // namespace mxe
