// Near field (P2P): exact regularised Biot-Savart velocity and gradient over
// the 27 adjacent leaves (paper Sec. 3.1, last paragraph; kernel eqs. 5-8).
//
// One target particle per lane.  Source particles are read at wave-uniform
// addresses, so they arrive through scalar loads and sit in SGPRs: every lane of
// the wave works on the same source at the same time.  The pair kernel, with
// r = x_i - x_j and rho = r/sigma:
//   q      = g(rho) / r^3,  g = erf(rho/sqrt2) - sqrt(2/pi) rho exp(-rho^2/2)
//   q'/r   = (sqrt(2/pi) sigma^-3 exp(-rho^2/2) - 3 q) / r^2
//   u     += q alpha_j x r
//   J[a][b] += (q'/r) r_a (alpha_j x r)_b + q eps_abc alpha_j,c
// For small rho both q and q'/r are even power series in rho (g is the
// integral of the Gaussian mass, g' = sqrt(2/pi) rho^2 exp(-rho^2/2)).
// A target block of 48 or fewer particles is split over lane groups that share
// out the sources.  The sums go to the near buffer that L2P combines with the
// far field, or, without one, through the epilogue here: far field, the
// gradient's contraction into the stretching term, the caller's order.
#include "leaf_sums.h"

namespace vmfmm {

namespace {

constexpr double kSqrt2OverPi = 0.79788456080286535587989211986876373;

// a_n = (-1/2)^n / (n! (2n+3)): g / rho^3 = sqrt(2/pi) sum a_n rho^{2n}
// Horner in t = rho^2 over n = 0..NTERM-1; h1 = 2 d(h0)/dt = sum 2 n a_n t^{n-1}.
template <typename T, int NTERM>
__device__ __forceinline__ void small_rho(T t, T &h0, T &h1) {
    static_assert(NTERM >= 3 && NTERM <= 14, "series length");
    constexpr double a[14] = {
        1.0 / 3.0,
        -0.5 / 5.0,
        0.25 / (2.0 * 7.0),
        -0.125 / (6.0 * 9.0),
        0.0625 / (24.0 * 11.0),
        -0.03125 / (120.0 * 13.0),
        0.015625 / (720.0 * 15.0),
        -0.0078125 / (5040.0 * 17.0),
        0.00390625 / (40320.0 * 19.0),
        -0.001953125 / (362880.0 * 21.0),
        0.0009765625 / (3628800.0 * 23.0),
        -0.00048828125 / (39916800.0 * 25.0),
        0.000244140625 / (479001600.0 * 27.0),
        -0.0001220703125 / (6227020800.0 * 29.0),
    };
    constexpr int top = NTERM - 1;
    T s0 = T(a[top]), s1 = T(2.0 * top * a[top]);
#pragma unroll
    for (int k = top - 1; k >= 1; --k) {
        s0 = s0 * t + T(a[k]);
        s1 = s1 * t + T(2.0 * k * a[k]);
    }
    h0 = s0 * t + T(a[0]);
    h1 = s1;
}

// FP64 pair kernel.  For rho < 0.75 the series (13 terms, truncation below
// 1e-16 relative).  Beyond, with x = rho/sqrt2 and E = exp(-rho^2/2),
//   g = erf(x) - sqrt(2/pi) rho E = 1 - E (erfcx(x) + sqrt(2/pi) rho),
// erfcx(x) = exp(x^2) erfc(x) from a polynomial in u(y), y = (x - c)/(x + c)
// (about 5e-16 relative; x is clamped at 6.5, where E < 5e-19 makes the term
// vanish in double), and E = 2^(r^2 ke) by range reduction and a degree-13
// polynomial.  Reciprocal and reciprocal square root: hardware estimates
// refined by two Newton steps.  Coefficients: gen_pair64_coeffs.py.
// generated by python -m paper_1110_2921_amd.gen_pair64_coeffs
constexpr int kExp2Deg = 13;
constexpr double kExp2C[] = {1.0, 0.69314718055994530942, 0.24022650695910071233, 0.055504108664821579953, 0.009618129107628477162, 0.0013333558146428443423, 0.00015403530393381609954, 0.00001525273380405984028, 1.3215486790144309488e-6, 1.0178086009239699727e-7, 7.0549116208011233299e-9, 4.4455382718708114976e-10, 2.5678435993488205142e-11, 1.3691488853904128881e-12};
constexpr double kErfcxMapC = 4.0;
constexpr double kErfcxXmax = 6.5;
constexpr double kErfcxYmid = -0.26389025173983907894;
constexpr double kErfcxInvYhalf = 1.9920894532798966399;
constexpr int kErfcxDeg = 17;
constexpr double kErfcxC[] = {0.22423572770292414676, -0.21014786434620323928, 0.10294920578508665075, -0.042656503629381491589, 0.014902444795601051759, -0.0043380449909054518515, 0.001025663029747490918, -0.00018654007531639407121, 0.00002259024331165582876, -7.3370476876062302707e-7, -3.3502768230615760572e-7, 6.0982847915142381289e-8, 7.6883230134258380755e-10, -1.558713275172138385e-9, 9.8346917112621498825e-11, 3.5733441967993213118e-11, -3.7696720135044547941e-12, -7.9638008832713648522e-13};

struct Consts64 {
    double inv_s2, thr2;
    double kx;         // 1 / (sigma sqrt2): x = kx r
    double ke;         // -log2(e) / (2 sigma^2)
    double ks;         // sqrt(2/pi) / sigma
    double kd, kd5;    // sqrt(2/pi) / sigma^3, / sigma^5
    // polynomial coefficients held in registers for the whole kernel: FP64
    // instructions take no 64-bit literal, so otherwise every use inside the
    // source loop re-creates its constant with a move
    double e2[kExp2Deg + 1];
    double ex[kErfcxDeg + 1];
};

__device__ __forceinline__ Consts64 consts64(double sigma) {
    const double is = 1.0 / sigma;
    Consts64 k;
    k.inv_s2 = is * is;
    k.thr2 = 0.5625 * sigma * sigma;
    k.kx = 0.70710678118654752440 * is;
    k.ke = -0.5 * 1.4426950408889634074 * is * is;
    k.ks = kSqrt2OverPi * is;
    k.kd = kSqrt2OverPi * is * is * is;
    k.kd5 = k.kd * is * is;
#pragma unroll
    for (int n = 0; n <= kExp2Deg; ++n) {
        k.e2[n] = kExp2C[n];
        asm volatile("" : "+v"(k.e2[n]));
    }
#pragma unroll
    for (int n = 0; n <= kErfcxDeg; ++n) {
        k.ex[n] = kErfcxC[n];
        asm volatile("" : "+v"(k.ex[n]));
    }
    return k;
}

__device__ __forceinline__ double rcp64(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    return fma(r, fma(-d, r, 1.0), r);
}

__device__ __forceinline__ double rsq64(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// 2^y for y <= 0 (underflows to 0)
__device__ __forceinline__ double exp2_neg(double y, const double *c) {
    const double kf = rint(fmax(y, -1100.0));
    const double f = y - kf;
    double p = c[kExp2Deg];
#pragma unroll
    for (int n = kExp2Deg - 1; n >= 0; --n) p = fma(p, f, c[n]);
    return ldexp(p, int(kf));
}

__device__ __forceinline__ double erfcx_poly(double x, const double *c) {
    const double xc = fmin(x, kErfcxXmax);
    const double y = (xc - kErfcxMapC) * rcp64(xc + kErfcxMapC);
    const double u = (y - kErfcxYmid) * kErfcxInvYhalf;
    double p = c[kErfcxDeg];
#pragma unroll
    for (int n = kErfcxDeg - 1; n >= 0; --n) p = fma(p, u, c[n]);
    return p;
}

__device__ __forceinline__ void pair64(double r2, const Consts64 &k, double &q, double &dq) {
    // as pair32: the far form on every lane, the series by a select when some
    // lane of the wave needs it (its far-form values, inf or NaN at r = 0, are discarded)
    const double rinv = rsq64(r2);
    const double r = r2 * rinv;
    const double e = exp2_neg(r2 * k.ke, k.e2);
    const double g = fma(-e, fma(k.ks, r, erfcx_poly(k.kx * r, k.ex)), 1.0);
    const double ir2 = rinv * rinv;
    q = g * rinv * ir2;
    dq = fma(k.kd, e, -3.0 * q) * ir2;
    const bool small = r2 < k.thr2;
    if (__builtin_expect(__any(small), 0)) {
        double h0, h1;
        small_rho<double, 13>(r2 * k.inv_s2, h0, h1);
        q = small ? k.kd * h0 : q;
        dq = small ? k.kd5 * h1 : dq;
    }
}

struct Consts32 {
    float inv_s2, thr2;
    float sg;          // sigma: 1/rho = sg / r
    float ke;          // -log2(e) / (2 sigma^2): exp(-rho^2/2) = 2^(ke r^2)
    float ks;          // sqrt(2/pi) / sigma: sqrt(2/pi) rho = ks r
    float kd;          // sqrt(2/pi) / sigma^3
    float kd5;         // sqrt(2/pi) / sigma^5
};

__device__ __forceinline__ Consts32 consts32(double sigma) {
    const double is = 1.0 / sigma;
    Consts32 k;
    k.inv_s2 = float(is * is);
    k.thr2 = float(sigma * sigma);
    k.sg = float(sigma);
    k.ke = float(-0.5 * 1.4426950408889634074 * is * is);
    k.ks = float(kSqrt2OverPi * is);
    k.kd = float(kSqrt2OverPi * is * is * is);
    k.kd5 = float(kSqrt2OverPi * is * is * is * is * is);
    return k;
}

// FP32 pair kernel.  For rho < 1 the series (9 terms, truncation < 1e-9
// relative) is used; beyond,
//   1 - g = exp(-rho^2/2) (E(1/rho) + sqrt(2/pi) rho),
// E a degree-6 polynomial in 1/rho for erfcx(rho/sqrt2) (weighted minimax fit,
// below 2e-7 relative error in g; the FP32 rounding of 1 - g, about 1e-6
// relative at rho = 1, is the larger error).  1/rho = sigma rinv comes from the
// reciprocal square root the pair needs anyway, so the far form takes two
// transcendentals (rsqrt, exp2), each issued at a quarter of the FMA rate, and
// no reciprocal.  The series branch diverges within a wave whenever one lane
// is close to the source, so its threshold is kept as small as that accuracy
// allows.  1/sigma is folded into the constants; the Gaussian is one hardware
// exp2 of r^2 ke.
// generated by python -m paper_1110_2921_amd.gen_pair32_coeffs (max relative error of g 1.8e-07 on rho in [1, 14])
constexpr int kErfcxDeg32 = 6;
constexpr float kErfcxU32[] = {-7.622858584e-03f, 8.803889779e-01f, -3.428088361e-01f, -2.458618671e-01f, 4.284188107e-01f, -2.400247991e-01f, 5.066721522e-02f};

__device__ __forceinline__ void pair32(float r2, const Consts32 &k, float &q, float &dq) {
    // Every lane takes the rho >= 1 form (no exec-mask branch per pair); when a
    // lane of the wave is below the threshold (wave-uniform test, rare) the
    // series replaces its values by a select (the first form's values there,
    // inf or NaN at r = 0, are discarded).
    const float rinv = __frsqrt_rn(r2);
    const float r = r2 * rinv;
    const float u = k.sg * rinv;
    const float e = __builtin_amdgcn_exp2f(r2 * k.ke);
    float ex = kErfcxU32[kErfcxDeg32];
#pragma unroll
    for (int i = kErfcxDeg32 - 1; i >= 0; --i) ex = fmaf(ex, u, kErfcxU32[i]);
    const float g = fmaf(-e, fmaf(k.ks, r, ex), 1.0f);
    const float ir2 = rinv * rinv;
    q = g * rinv * ir2;
    dq = fmaf(k.kd, e, -3.0f * q) * ir2;
    const bool small = r2 < k.thr2;
    if (__builtin_expect(__any(small), 0)) {
        float h0, h1;
        small_rho<float, 9>(r2 * k.inv_s2, h0, h1);
        q = small ? k.kd * h0 : q;
        dq = small ? k.kd5 * h1 : dq;
    }
}

// The pair function from a table.  With t = rho^2 = r^2 / sigma^2,
//   q = Q(t) / sigma^3,  q'/r = 2 Q'(t) / sigma^5,  Q(t) = g / rho^3:
// both are one smooth function of t and its derivative, so one polynomial
// serves both (Horner with the derivative alongside), without a reciprocal
// square root, an exponential or erfc per pair.  Rows are segments of t, 2^SEG
// per octave from 2^kPairTabLo to 2^kPairTabHi (index: the exponent and the top
// mantissa bits of t) and row 0 for [0, 2^kPairTabLo); a row holds the
// coefficients of Q in x = t - c, c the segment's centre, chosen so that 2 Q'
// is the truncated Chebyshev series of q'/r (host, extended precision).  From
// t = 2^kPairTabHi on g is 1 and Q = t^-3/2: t is scaled by 4^-e into the last
// two octaves and the results by 8^-e and 32^-e.
// FP64: 64 segments per octave, degree 7, largest relative error against
// 40-digit arithmetic 2.1e-16 in q and 7.0e-16 in q'/r (the polynomial erfc and
// exponential of pair64: 3.2e-15 and 2.9e-14); FP32: 32 per octave, degree 4,
// 1.0e-7 and 1.6e-7 (pair32: 5.9e-7 and 3.5e-6).
// The table (FP64 57 KB, FP32 9 KB) sits in LDS in planes of 16 bytes per row,
// so that the lanes' rows spread over the banks (a 16-byte gather of 64 lanes
// takes 14 cycles, 4 of them without conflicts).
// FP64: 50 instead of 97 FP64 instructions a pair at 4 instead of 2 waves per
// SIMD, 8.0 instead of 13.3 ms at 128^3 (350 cycles a wave and source, of which
// VALU 215 and LDS 221 of the CU's); FP32: 25.9 against 26.2 ms at 256^3, LDS
// gathers for what the two transcendentals took.
typedef double dbl2 __attribute__((ext_vector_type(2)));
typedef float flt4 __attribute__((ext_vector_type(4)));

typedef const __attribute__((address_space(3))) char *LdsBytes;

template <typename T> struct PairTab;
template <> struct PairTab<double> {
    typedef dbl2 Vec;   // 16 bytes
    static constexpr int seg = kPairSeg64, rows = pair_rows(kPairSeg64);
    static constexpr int bytes = rows * 8 * kPairCoefs64;
    static constexpr int mant = 20, bias = 1023;   // of the high word
    static __device__ __forceinline__ int word(double t) { return __double2hiint(t); }
    static __device__ __forceinline__ double real(int w) { return __hiloint2double(w, 0); }
    static __device__ __forceinline__ double with(double t, int w) { return __hiloint2double(w, __double2loint(t)); }
    struct Row {
        dbl2 c01, c23, c45, c67;
    };
    static __device__ __forceinline__ Row load(LdsBytes row) {
        typedef const __attribute__((address_space(3))) dbl2 *P;
        const P c = (P)row;
        return {c[0], c[rows], c[2 * rows], c[3 * rows]};
    }
    static __device__ __forceinline__ void eval(const Row &r, double x, double &Q, double &H) {
        const dbl2 c01 = r.c01, c23 = r.c23, c45 = r.c45, c67 = r.c67;
        double d = c67.y, p = fma(c67.y, x, c67.x);
        d = fma(d, x, p); p = fma(p, x, c45.y);
        d = fma(d, x, p); p = fma(p, x, c45.x);
        d = fma(d, x, p); p = fma(p, x, c23.y);
        d = fma(d, x, p); p = fma(p, x, c23.x);
        d = fma(d, x, p); p = fma(p, x, c01.y);
        Q = fma(p, x, c01.x);
        H = fma(d, x, p);
    }
    static __device__ __forceinline__ double scale(double v, int e) { return ldexp(v, e); }
};
template <> struct PairTab<float> {
    typedef flt4 Vec;
    static constexpr int seg = kPairSeg32, rows = pair_rows(kPairSeg32);
    static constexpr int bytes = rows * 16 * 2;
    static constexpr int mant = 23, bias = 127;
    static __device__ __forceinline__ int word(float t) { return __float_as_int(t); }
    static __device__ __forceinline__ float real(int w) { return __int_as_float(w); }
    static __device__ __forceinline__ float with(float, int w) { return __int_as_float(w); }
    struct Row {
        flt4 c0;
        float c4;
    };
    static __device__ __forceinline__ Row load(LdsBytes row) {
        typedef const __attribute__((address_space(3))) flt4 *P;
        const P c = (P)row;
        return {c[0], ((const __attribute__((address_space(3))) float *)(c + rows))[0]};
    }
    static __device__ __forceinline__ void eval(const Row &r, float x, float &Q, float &H) {
        const flt4 c0 = r.c0;
        const float c4 = r.c4;
        float d = c4, p = fmaf(c4, x, c0.w);
        d = fmaf(d, x, p); p = fmaf(p, x, c0.z);
        d = fmaf(d, x, p); p = fmaf(p, x, c0.y);
        Q = fmaf(p, x, c0.x);
        H = fmaf(d, x, p);
    }
    static __device__ __forceinline__ float scale(float v, int e) { return ldexpf(v, e); }
};

// exponent e that brings t below the table's end (0 within the table)
template <typename T>
__device__ __forceinline__ int table_shift(T t) {
    using P = PairTab<T>;
    const int w = P::word(t);
    return w >= ((P::bias + kPairTabHi) << P::mant) ? ((w >> P::mant) - (P::bias + kPairTabHi - 2)) >> 1 : 0;
}

// t's row, and x = t - c
template <typename T>
__device__ __forceinline__ LdsBytes table_row(T t, uint32_t tab, T &x) {
    using P = PairTab<T>;
    constexpr int sh = P::mant - P::seg;
    constexpr int lo = ((P::bias + kPairTabLo) << P::seg) - 1, hi = lo + P::rows - 1;
    int idx = P::word(t) >> sh;
    idx = idx < lo ? lo : (idx > hi ? hi : idx);
    x = t - P::real((idx << sh) | (1 << (sh - 1)));
    // one LDS address (the table's, less its first row's index, in `tab`), the
    // planes at immediate offsets from it
    uint32_t at = (uint32_t(idx) << 4) + tab;
    asm("" : "+v"(at));
    return (LdsBytes)at;
}
// what table_row takes for a table at LDS address `at`
template <typename T>
__device__ __forceinline__ uint32_t table_base(uint32_t at) {
    using P = PairTab<T>;
    return at - 16u * uint32_t(((P::bias + kPairTabLo) << P::seg) - 1);
}

// Q and Q' (H) of NS pairs at squared distances r2
template <int NS, typename T>
__device__ __forceinline__ void table_pairs(const T (&r2)[NS], T inv_s2, uint32_t tab, T (&q)[NS], T (&h)[NS]) {
    using P = PairTab<T>;
    T t[NS];
    int w = 0;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        t[i] = r2[i] * inv_s2;
        w = max(w, P::word(t[i]));
    }
    // beyond the table (wave-uniform test, rare): t scaled down before, the results after
    const bool beyond = __builtin_amdgcn_ballot_w64(w >= ((P::bias + kPairTabHi) << P::mant)) != 0;
    if (__builtin_expect(beyond, 0)) {
#pragma unroll
        for (int i = 0; i < NS; ++i) t[i] = P::with(t[i], P::word(t[i]) - (table_shift(t[i]) << (P::mant + 1)));
    }
    // every row's reads issued before the first polynomial
    typename P::Row row[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) row[i] = P::load(table_row(t[i], tab, t[i]));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NS; ++i) P::eval(row[i], t[i], q[i], h[i]);
    if (__builtin_expect(beyond, 0)) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int e = table_shift(r2[i] * inv_s2);
            q[i] = P::scale(q[i], -3 * e);
            h[i] = P::scale(h[i], -5 * e);
        }
    }
}

// One precision's pair arithmetic.  TAB: the pair function from the table, in
// units of sigma (the sums are scaled by cu = 1/sigma^3 and cj = 2/sigma^5 at the
// end); else pair64 / pair32, the form for cores so small beside the leaf that
// those units would leave the type's range (launch_p2p*).
template <bool TAB>
struct Pol64 {
    using Rec = Part64;
    using Real = double;
    uint32_t tab;
    double inv_s2, cu, cj;
    Consts64 k;
    struct Acc {
        double u[3], J[9], S[3];
    };
    static __device__ __forceinline__ Real scaled(Real x) { return x; }
    static __device__ __forceinline__ void clear(Acc &A) {
#pragma unroll
        for (int c = 0; c < 3; ++c) A.u[c] = A.S[c] = 0.0;
#pragma unroll
        for (int c = 0; c < 9; ++c) A.J[c] = 0.0;
    }
    __device__ __forceinline__ Pol64(double sigma, uint32_t table) : tab(table), inv_s2(0.0), cu(1.0), cj(1.0) {
        if constexpr (TAB) {
            const double is = 1.0 / sigma;
            inv_s2 = is * is;
            cu = is * is * is;
            cj = 2.0 * cu * inv_s2;
        } else {
            k = consts64(sigma);
        }
    }
    __device__ __forceinline__ void add(const Part64 &s, const double (&r)[3], double q, double h, Acc &A) const {
        const double c0 = s.ay * r[2] - s.az * r[1];
        const double c1 = s.az * r[0] - s.ax * r[2];
        const double c2 = s.ax * r[1] - s.ay * r[0];
        A.u[0] += q * c0;
        A.u[1] += q * c1;
        A.u[2] += q * c2;
        A.S[0] += q * s.ax;
        A.S[1] += q * s.ay;
        A.S[2] += q * s.az;
        const double t0 = h * c0, t1 = h * c1, t2 = h * c2;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            A.J[3 * i] += r[i] * t0;
            A.J[3 * i + 1] += r[i] * t1;
            A.J[3 * i + 2] += r[i] * t2;
        }
    }
    // NS sources at once (one test for pairs beyond the table)
    template <int NS>
    __device__ __forceinline__ void pairs(const Part64 *__restrict__ src, double tx, double ty, double tz,
                                          Acc &A) const {
        Part64 s[NS];
        double r[NS][3], r2[NS], q[NS], h[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            s[i] = src[i];
            r[i][0] = tx - s[i].dx;
            r[i][1] = ty - s[i].dy;
            r[i][2] = tz - s[i].dz;
            r2[i] = r[i][0] * r[i][0] + r[i][1] * r[i][1] + r[i][2] * r[i][2];
        }
        if constexpr (TAB) {
            table_pairs<NS, double>(r2, inv_s2, tab, q, h);
        } else {
#pragma unroll
            for (int i = 0; i < NS; ++i) pair64(r2[i], k, q[i], h[i]);
        }
#pragma unroll
        for (int i = 0; i < NS; ++i) add(s[i], r[i], q[i], h[i], A);
    }
    __device__ __forceinline__ void uniform(const Part64 *__restrict__ parts, int js, int je, double tx, double ty,
                                            double tz, Acc &A) const {
        constexpr int NS = TAB ? 2 : 1;
        int j = js;
        for (; j + NS <= je; j += NS) pairs<NS>(parts + j, tx, ty, tz, A);
        if (NS > 1 && j < je) pairs<1>(parts + j, tx, ty, tz, A);
    }
    __device__ __forceinline__ void grouped(const Part64 *__restrict__ parts, int js, int je, int ng, double tx,
                                            double ty, double tz, Acc &A) const {
#pragma unroll 1
        for (int j = js; j < je; j += ng) pairs<1>(parts + j, tx, ty, tz, A);
    }
    // row K of the near sums
    template <int K>
    __device__ __forceinline__ double value(const Acc &A) const {
        if constexpr (K < 3) return A.u[K] * cu;
        else if constexpr (K < 12) return A.J[K - 3] * cj;
        else return A.S[K - 12] * cu;
    }
};

// Mixed precision: FP32 pair arithmetic.  Velocity sums: each block of at most
// kKahanBlock consecutive sources is summed plainly in FP32 (up), and the block
// sums enter the running total through Kahan's compensated addition (us, uc).
// Per pair that is one FMA per component instead of a compensated step (4
// instructions), and the rounding left is that of 16-term FP32 sums, around
// 1e-7 of the block's terms.
constexpr int kKahanBlock = 16;

// FP32 table: Q and Q' times 2^fold.  A term in units of sigma, Q' (alpha x r) r, has
// the magnitude sigma^5 alpha / r^3, which leaves FP32's range for cores far below
// the leaf or small units long before alpha / r^3 does; about sigma^-4 more and the
// velocity's and the gradient's terms are within a factor sigma of those in physical
// units.  A power of two: no result in range changes.  The limits keep the
// coefficients normal (largest 0.27, smallest that counts 2^-60).
__device__ __forceinline__ int fold32(double sigma) { return min(100, max(-64, -4 * ilogb(sigma))); }

template <bool TAB>
struct Pol32 {
    using Rec = Part32;
    using Real = float;
    uint32_t tab;
    float inv_s2;
    double cu, cj;
    Consts32 k;
    struct Acc {
        float us[3], uc[3], up[3], J[9], S[3];
    };
    static __device__ __forceinline__ Real scaled(Real x) { return x; }
    static __device__ __forceinline__ void clear(Acc &A) {
#pragma unroll
        for (int c = 0; c < 3; ++c) A.us[c] = A.uc[c] = A.up[c] = A.S[c] = 0.0f;
#pragma unroll
        for (int c = 0; c < 9; ++c) A.J[c] = 0.0f;
    }
    __device__ __forceinline__ Pol32(double sigma, uint32_t table) : tab(table), inv_s2(0.0f), cu(1.0), cj(1.0) {
        if constexpr (TAB) {
            const double is = 1.0 / sigma;
            inv_s2 = float(is * is);
            cu = ldexp(is * is * is, -fold32(sigma));
            cj = 2.0 * cu * is * is;
        } else {
            k = consts32(sigma);
        }
    }
    static __device__ __forceinline__ void flush(Acc &A) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const float y = A.up[b] - A.uc[b];
            const float t = A.us[b] + y;
            A.uc[b] = (t - A.us[b]) - y;
            A.us[b] = t;
            A.up[b] = 0.0f;
        }
    }
    template <int NS>
    __device__ __forceinline__ void pairs(const Part32 *__restrict__ src, float tx, float ty, float tz,
                                          Acc &A) const {
        Part32 s[NS];
        float r[NS][3], r2[NS], q[NS], h[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            s[i] = src[i];
            r[i][0] = tx - s[i].dx;
            r[i][1] = ty - s[i].dy;
            r[i][2] = tz - s[i].dz;
            r2[i] = r[i][0] * r[i][0] + r[i][1] * r[i][1] + r[i][2] * r[i][2];
        }
        if constexpr (TAB) {
            table_pairs<NS, float>(r2, inv_s2, tab, q, h);
        } else {
#pragma unroll
            for (int i = 0; i < NS; ++i) pair32(r2[i], k, q[i], h[i]);
        }
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const float c[3] = {s[i].ay * r[i][2] - s[i].az * r[i][1], s[i].az * r[i][0] - s[i].ax * r[i][2],
                                s[i].ax * r[i][1] - s[i].ay * r[i][0]};
#pragma unroll
            for (int b = 0; b < 3; ++b) A.up[b] = fmaf(q[i], c[b], A.up[b]);
            A.S[0] += q[i] * s[i].ax;
            A.S[1] += q[i] * s[i].ay;
            A.S[2] += q[i] * s[i].az;
            const float t0 = h[i] * c[0], t1 = h[i] * c[1], t2 = h[i] * c[2];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                A.J[3 * d] += r[i][d] * t0;
                A.J[3 * d + 1] += r[i][d] * t1;
                A.J[3 * d + 2] += r[i][d] * t2;
            }
        }
    }
    __device__ __forceinline__ void uniform(const Part32 *__restrict__ parts, int js, int je, float tx, float ty,
                                            float tz, Acc &A) const {
        for (int jb = js; jb < je; jb += kKahanBlock) {
            const int jend = min(jb + kKahanBlock, je);
            int j = jb;
            for (; j + 4 <= jend; j += 4) pairs<4>(parts + j, tx, ty, tz, A);
            for (; j < jend; ++j) pairs<1>(parts + j, tx, ty, tz, A);
            flush(A);
        }
    }
    __device__ __forceinline__ void grouped(const Part32 *__restrict__ parts, int js, int je, int ng, float tx,
                                            float ty, float tz, Acc &A) const {
        // this lane group takes every ng-th source: blocks of kKahanBlock of its own sources
        for (int jb = js; jb < je; jb += ng * kKahanBlock) {
            const int jend = min(jb + ng * kKahanBlock, je);
#pragma unroll 1
            for (int j = jb; j < jend; j += ng) pairs<1>(parts + j, tx, ty, tz, A);
            flush(A);
        }
    }
    template <int K>
    __device__ __forceinline__ double value(const Acc &A) const {
        if constexpr (K < 3) return (double(A.us[K]) - double(A.uc[K])) * cu;
        else if constexpr (K < 12) return double(A.J[K - 3]) * cj;
        else return double(A.S[K - 12]) * cu;
    }
};

// Copies the table (FP32: folded) to the start of the dynamic LDS; what the policies
// take for it.
template <typename T, bool TAB>
__device__ __forceinline__ uint32_t load_table(const P2PArgs &a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if constexpr (TAB) {
        typedef typename PairTab<T>::Vec V;
        const V *src = reinterpret_cast<const V *>(a.table);
        V *dst = reinterpret_cast<V *>(smem_raw);
        const T f = sizeof(T) == 4 ? ldexp(T(1), fold32(a.sigma)) : T(1);
        for (int i = threadIdx.x; i < PairTab<T>::bytes / 16; i += kP2PThreads) dst[i] = src[i] * f;
        __syncthreads();
    }
    return table_base<T>(uint32_t(uintptr_t((LdsBytes)smem_raw)));
}

template <class POL, bool SPLIT, bool TAB>
__device__ __forceinline__ void p2p_body(const P2PArgs &a, const typename POL::Rec *__restrict__ parts) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    using T = typename POL::Real;
    p2p_leaves<POL, SPLIT>(a, parts, POL(a.sigma, load_table<T, TAB>(a)),
                           reinterpret_cast<double *>(smem_raw + (TAB ? PairTab<T>::bytes : 0)));
}

template <bool SPLIT, bool TAB>
__global__ void __launch_bounds__(kP2PThreads) __attribute__((amdgpu_waves_per_eu(TAB ? 4 : 2, TAB ? 4 : 2)))
k_p2p64(P2PArgs a, const Part64 *__restrict__ parts) {
    p2p_body<Pol64<TAB>, SPLIT, TAB>(a, parts);
}

template <bool SPLIT, bool TAB>
__global__ void __launch_bounds__(kP2PThreads) __attribute__((amdgpu_waves_per_eu(6, 6)))
k_p2p32(P2PArgs a, const Part32 *__restrict__ parts) {
    p2p_body<Pol32<TAB>, SPLIT, TAB>(a, parts);
}

// Adaptive tree: work item w is the target block items[w] = (leaf i in particle
// order, first target of the block of up to 64 within the leaf), its sources the
// leaf's P2P list: entry (source range, D = centre_b + s L - centre_a) contributes
// x_i - x_j - s L = (delta_i - D) - delta_j, the records relative to their own
// leaf centres.  Items differ by a factor of ten in work and a workgroup's table
// and registers hold half a compute unit, so the workgroups are as many as fit and
// take items one by one, first from their XCD's contiguous eighth (neighbour
// leaves share its L2), then from the others' (ctr[8]: items taken of each eighth,
// zero at the start).  Wave w takes entries w, w + 8, ... of the item's list, the
// waves' sums added in wave order: a wave per item ended with the longest item
// (20011 particles in leaves of 32: 400 us, the evaluation 1.64 ms, now 1.36; 2^17
// in leaves of 64 4.09 and 3.58; 2^19 no difference).  P2P of 2^19 clustered
// particles 2.05 ms (pair function by polynomials: 3.83 ms).
template <bool TAB>
__global__ void __launch_bounds__(kP2PThreads) __attribute__((amdgpu_waves_per_eu(TAB ? 4 : 2, TAB ? 4 : 2)))
k_p2p64_list(P2PArgs a, int nitem, const int2 *__restrict__ items, const int32_t *__restrict__ lcell,
             const int32_t *__restrict__ lstart, const uint32_t *__restrict__ off, const uint32_t *__restrict__ cnt,
             const P2PMeta *__restrict__ meta, const Part64 *__restrict__ parts, int *__restrict__ ctr) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ int taken;
    const Pol64<TAB> pol(a.sigma, load_table<double, TAB>(a));
    double *red = reinterpret_cast<double *>(smem_raw + (TAB ? PairTab<double>::bytes : 0));
    double *fin = red + kRedRows * kP2PThreads;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int k = 0; k < 8; ++k) {
        const int x = int(blockIdx.x + k) & 7;
        const int i0 = int(int64_t(nitem) * x / 8), ni = int(int64_t(nitem) * (x + 1) / 8) - i0;
        for (;;) {
            if (tid == 0) taken = atomicAdd(&ctr[x], 1);
            __syncthreads();
            const int w = __builtin_amdgcn_readfirstlane(taken);
            __syncthreads();
            if (w >= ni) break;
            const int2 it = items[i0 + w];
            const int c = lcell[it.x];
            const int s0 = lstart[it.x], end = min(lstart[it.x + 1] - s0, it.y + 64);
            const uint32_t e0 = off[c] + uint32_t(wave), e1 = off[c] + cnt[c];
            for (int base = it.y; base < end;) {
                const int E = piece_lanes(end - base), b0 = base;
                base += E;
                const int t = lane & (E - 1), grp = lane / E, ng = 64 / E;
                const bool write = b0 + t < end && grp == 0;
                const int gi = s0 + (b0 + t < end ? b0 + t : b0);
                const Part64 me = parts[gi];
                typename Pol64<TAB>::Acc A;
                Pol64<TAB>::clear(A);
                // the next entry's record is fetched while the current one's sources are evaluated
                P2PMeta mn{};
                if (e1 > e0) mn = meta[e0];
                for (uint32_t e = e0; e < e1; e += kP2PWaves) {
                    const P2PMeta m = mn;
                    mn = meta[e + kP2PWaves < e1 ? e + kP2PWaves : e];
                    const double tx = me.dx - m.dx, ty = me.dy - m.dy, tz = me.dz - m.dz;
                    if (E == 64) pol.uniform(parts, m.js, m.je, tx, ty, tz, A);
                    else pol.grouped(parts, m.js + grp, m.je, ng, tx, ty, tz, A);
                }
                auto value = [&](auto kc) { return pol.template value<decltype(kc)::value>(A); };
                for_rows([&](auto rc) {
                    wave_round<decltype(rc)::value>(red, value,
                                                    [&](int r, double v) { fin[r * 64 + lane] = group_sum(v, E); });
                }, std::make_integer_sequence<int, kNearRows / kRedRows>{});
                if (wave == 0) finish(a, gi, write, [&](int r) { return fin[64 * r + lane]; });
            }
        }
    }
}

template <typename R>
using P2PKernel = void (*)(P2PArgs, const R *);

}  // namespace

// workgroups the chip holds at once (80 / 128 registers per lane)
static int p2p_slots(bool mixed) { return compute_units() * (mixed ? 3 : 2); }

// Shares that fill the chip, but no fewer than 16 sources a wave: a share costs a
// copy of the table and a term of every L2P sum (768 particles at level 2 in FP64:
// 26 us with 2 shares, 34 with 8).
int p2p_shares(int nleaf, int ntarget, int nsource, bool mixed) {
    const int slots = p2p_slots(mixed);
    const int64_t per_wave = int64_t(27) * nsource / nleaf / kP2PWaves;
    const int most = int(std::min<int64_t>(kP2PMaxShares, per_wave / 16));
    return std::max(1, std::min(most, slots / (nleaf * p2p_blocks(nleaf, ntarget, slots))));
}

// The table needs sigma-unit distances, their powers t^-3/2 and t^-5/2 (the terms
// that these enter: fold32) and, in FP32, 1/sigma^2 within the type's range.
hipError_t launch_p2p64(hipStream_t s, const P2PArgs &a, const Part64 *parts) {
    const bool tab = a.sigma >= 0x1p-100 * a.w;
    const P2PShape p = p2p_shape(a, p2p_slots(false), tab ? PairTab<double>::bytes : 0);
    const P2PKernel<Part64> k = p.split ? (tab ? k_p2p64<true, true> : k_p2p64<true, false>)
                                        : (tab ? k_p2p64<false, true> : k_p2p64<false, false>);
    hipLaunchKernelGGL(k, p.grid, dim3(kP2PThreads), p.smem, s, a, parts);
    return hipGetLastError();
}

hipError_t launch_p2p32(hipStream_t s, const P2PArgs &a, const Part32 *parts) {
    const bool tab = a.sigma >= 0x1p-20 * a.w && a.sigma >= 0x1p-50 && a.sigma <= 0x1p50;
    const P2PShape p = p2p_shape(a, p2p_slots(true), tab ? PairTab<float>::bytes : 0);
    const P2PKernel<Part32> k = p.split ? (tab ? k_p2p32<true, true> : k_p2p32<true, false>)
                                        : (tab ? k_p2p32<false, true> : k_p2p32<false, false>);
    hipLaunchKernelGGL(k, p.grid, dim3(kP2PThreads), p.smem, s, a, parts);
    return hipGetLastError();
}

hipError_t launch_p2p64_list(hipStream_t s, const P2PArgs &a, int nitem, const int2 *items, const int32_t *lcell,
                             const int32_t *lstart, const uint32_t *off, const uint32_t *cnt, const P2PMeta *meta,
                             const Part64 *parts, int *ctr) {
    if (nitem == 0) return hipSuccess;
    // a.w: the root's width, the largest a leaf can have
    const bool tab = a.sigma >= 0x1p-100 * a.w;
    const int wgs = std::min(p2p_slots(false), nitem);
    const auto k = tab ? k_p2p64_list<true> : k_p2p64_list<false>;
    const size_t smem = (tab ? PairTab<double>::bytes : 0) + sizeof(double) * kRedDoubles;
    hipLaunchKernelGGL(k, dim3(unsigned(wgs)), dim3(kP2PThreads), smem, s, a, nitem, items, lcell, lstart, off, cnt,
                       meta, parts, ctr);
    return hipGetLastError();
}

}  // namespace vmfmm
