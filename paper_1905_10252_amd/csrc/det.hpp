// Deterministic arithmetic used wherever a floating-point result decides an
// integer or feeds a bit-exact particle trajectory.  Every function is a fixed
// sequence of IEEE-754 binary64 operations (add, mul, fma, div, sqrt, rint,
// ldexp, frexp), so the device and any other faithful implementation of the
// same sequence agree bit for bit.  Compiled without FP contraction.
//
//   det_exp : Cody-Waite reduction x = k ln2 + r with the fdlibm two-part ln 2,
//             then e^r by its Taylor polynomial of degree 13 (Horner, fma),
//             then ldexp by k.
//   det_log : x = m 2^e with m in [sqrt(1/2), sqrt(2)); log m = 2 atanh(f),
//             f = (m - 1)/(m + 1), odd series through f^23 (Horner in f^2,
//             fma); result e ln2_hi + (e ln2_lo + log m) with fma.
//   det_atan: |z| > 1 folded by atan z = pi/2 - atan(1/z); two halvings
//             a <- a / (1 + sqrt(1 + a^2)) (atan a = 2 atan of the result);
//             odd Taylor series of atan to a^25 by Horner in a^2 with fma;
//             times 4; pi/2 as a two-part constant.
//   Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) and standard normals by
//   the Marsaglia-Bray polar method on its 53-bit uniforms.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace smc {

// Constants of the polynomials.  An FP64 vector instruction cannot carry a
// 64-bit immediate, and left alone the compiler rebuilds every coefficient in
// vector registers (two v_mov_b32 a use: 4.8 cycles beside the 5 of a
// v_fma_f64) or, where a loop encloses the use, keeps all of them in scalar
// registers and spills those into vector lanes.  Scalar moves are no way out:
// the CU issues one a cycle for its four SIMDs, and two to each fma measured 9.3
// cycles a coefficient.  So the coefficients sit in constant memory and each
// evaluation reads its table with one or two wide scalar loads; the address
// passes through an empty asm so that the reads stay at the evaluation.
typedef __attribute__((address_space(4))) double cdouble;

static __device__ __constant__ const double kExpTab[14] = {
    0x1.71547652b82fep+0,   // log2 e
    0x1.62e42fee00000p-1,   // ln 2, high and low part
    0x1.a39ef35793c76p-33,
    0x1.6124613a86d09p-33,  // 1/13!
    0x1.1eed8eff8d898p-29,  // 1/12!
    0x1.ae64567f544e4p-26,  // 1/11!
    0x1.27e4fb7789f5cp-22,  // 1/10!
    0x1.71de3a556c734p-19,  // 1/9!
    0x1.a01a01a01a01ap-16,  // 1/8!
    0x1.a01a01a01a01ap-13,  // 1/7!
    0x1.6c16c16c16c17p-10,  // 1/6!
    0x1.1111111111111p-7,   // 1/5!
    0x1.5555555555555p-5,   // 1/4!
    0x1.5555555555555p-3,   // 1/3!
};

static __device__ __constant__ const double kLogTab[13] = {
    0x1.642c8590b2164p-4,   // 2/23
    0x1.8618618618618p-4,   // 2/21
    0x1.af286bca1af28p-4,   // 2/19
    0x1.e1e1e1e1e1e1ep-4,   // 2/17
    0x1.1111111111111p-3,   // 2/15
    0x1.3b13b13b13b14p-3,   // 2/13
    0x1.745d1745d1746p-3,   // 2/11
    0x1.c71c71c71c71cp-3,   // 2/9
    0x1.2492492492492p-2,   // 2/7
    0x1.999999999999ap-2,   // 2/5
    0x1.5555555555555p-1,   // 2/3
    0x1.a39ef35793c76p-33,  // ln 2, low and high part
    0x1.62e42fee00000p-1,
};

static __device__ __constant__ const double kAtanTab[12] = {
    0x1.47ae147ae147bp-5,   // 1/25
    0x1.642c8590b2164p-5,   // 1/23
    0x1.8618618618618p-5,   // 1/21
    0x1.af286bca1af28p-5,   // 1/19
    0x1.e1e1e1e1e1e1ep-5,   // 1/17
    0x1.1111111111111p-4,   // 1/15
    0x1.3b13b13b13b14p-4,   // 1/13
    0x1.745d1745d1746p-4,   // 1/11
    0x1.c71c71c71c71cp-4,   // 1/9
    0x1.2492492492492p-3,   // 1/7
    0x1.999999999999ap-3,   // 1/5
    0x1.5555555555555p-2,   // 1/3
};

template <int N>
__device__ inline const cdouble *coef_table(const double (&tab)[N])
{
    const cdouble *p = (const cdouble *)&tab[0];
    asm volatile("" : "+s"(p));
    return p;
}

// fma(p, v, c) with c read as a scalar operand (written out: for a lone chain
// the compiler would copy c into vector registers to use the two-operand form).
__device__ inline double fma_sc(double p, double v, double c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(p), "v"(v), "s"(c));
    return r;
#else
    return fma(p, v, c);
#endif
}

#define SMC_EACH for (int w = 0; w < W; ++w)

// a / b for positive b and quotients, both far from the ends of the exponent
// range (|a|, |b| and |a / b| within 2^-900 .. 2^900, or a = 0): the compiler's
// sequence (reciprocal, two Newton steps, quotient, residual) without the
// operand scaling and fix-up that only such ends need; correctly rounded, so
// the same bits as the operator.  8 instructions instead of 11.
template <int W>
__device__ inline void det_div_w(const double (&a)[W], const double (&b)[W], double (&q)[W])
{
    double y[W], e[W];
#pragma unroll
    SMC_EACH y[w] = __builtin_amdgcn_rcp(b[w]);
#pragma unroll
    SMC_EACH e[w] = fma(-b[w], y[w], 1.0);
#pragma unroll
    SMC_EACH y[w] = fma(y[w], e[w], y[w]);
#pragma unroll
    SMC_EACH e[w] = fma(-b[w], y[w], 1.0);
#pragma unroll
    SMC_EACH y[w] = fma(y[w], e[w], y[w]);
#pragma unroll
    SMC_EACH e[w] = a[w] * y[w];
#pragma unroll
    SMC_EACH q[w] = fma(fma(-b[w], e[w], a[w]), y[w], e[w]);
}

// sqrt(x) for x within 2^-700 .. 2^900: reciprocal root and Goldschmidt steps
// with two residual corrections, correctly rounded; without the scaling of
// small operands and the selects for 0 and infinity.
template <int W>
__device__ inline void det_sqrt_w(const double (&x)[W], double (&r)[W])
{
    double g[W], h[W], e[W];
#pragma unroll
    SMC_EACH {
        const double y = __builtin_amdgcn_rsq(x[w]);
        g[w] = x[w] * y;
        h[w] = y * 0.5;
    }
#pragma unroll
    SMC_EACH e[w] = fma(-h[w], g[w], 0.5);
#pragma unroll
    SMC_EACH {
        g[w] = fma(g[w], e[w], g[w]);
        h[w] = fma(h[w], e[w], h[w]);
    }
#pragma unroll
    SMC_EACH e[w] = fma(-g[w], g[w], x[w]);
#pragma unroll
    SMC_EACH g[w] = fma(e[w], h[w], g[w]);
#pragma unroll
    SMC_EACH e[w] = fma(-g[w], g[w], x[w]);
#pragma unroll
    SMC_EACH r[w] = fma(e[w], h[w], g[w]);
}


// e^x for x <= 709; 0 for NaN (every caller has flagged a NaN weight before).
template <int W>
__device__ inline void det_exp_w(const double (&x)[W], double (&y)[W])
{
    const cdouble *c = coef_table(kExpTab);
    double kd[W], r[W], p[W];
#pragma unroll
    SMC_EACH {
        r[w] = fmax(x[w], -746.0);  // e^-746 rounds to 0 in the ldexp below
        kd[w] = rint(r[w] * c[0]);
        r[w] = fma(-kd[w], c[1], r[w]);
    }
#pragma unroll
    SMC_EACH {
        r[w] = fma(-kd[w], c[2], r[w]);
        p[w] = c[3];
    }
#pragma unroll
    for (int k = 4; k < 14; ++k)
#pragma unroll
        SMC_EACH p[w] = fma_sc(p[w], r[w], c[k]);
#pragma unroll
    SMC_EACH {
        p[w] = fma(p[w], r[w], 0.5);  // 1/2!, 1/1!, 1/0!
        p[w] = fma(p[w], r[w], 1.0);
        p[w] = fma(p[w], r[w], 1.0);
        y[w] = ldexp(p[w], (int)kd[w]);
    }
}

__device__ inline double det_exp(double x)
{
    const double a[1] = {x};
    double y[1];
    det_exp_w<1>(a, y);
    return y[0];
}

// log x for normal positive x; kEnds: also +inf (itself) and NaN (NaN).
template <int W, bool kEnds = false>
__device__ inline void det_log_w(const double (&x)[W], double (&y)[W])
{
    const cdouble *c = coef_table(kLogTab);
    double f[W], s[W], p[W], q[W];
    int e[W];
#pragma unroll
    SMC_EACH {
        // x = m 2^e with m in [sqrt(1/2), sqrt(2)): the bits of x less those of
        // the lower end split into e (high 12 bits) and what m keeps
        constexpr uint64_t kLow = 0x3FE6A09E667F3BCDull;  // sqrt(1/2), rounded up
        const uint64_t b = (uint64_t)__double_as_longlong(x[w]);
        int top = (int)((b - kLow) >> 32);
        asm("" : "+v"(top));  // keeps the next lines in 32 bits
        e[w] = top >> 20;
        int hi = (int)(uint32_t)(b >> 32) - (top & (int)0xFFF00000);
        asm("" : "+v"(hi));
        const double m = __hiloint2double(hi, (int)(uint32_t)b);
        p[w] = m - 1.0;
        q[w] = m + 1.0;
    }
    det_div_w<W>(p, q, f);
#pragma unroll
    SMC_EACH {
        s[w] = f[w] * f[w];
        p[w] = c[0];
    }
#pragma unroll
    for (int k = 1; k < 11; ++k)
#pragma unroll
        SMC_EACH p[w] = fma_sc(p[w], s[w], c[k]);
#pragma unroll
    SMC_EACH {
        p[w] = fma(p[w], s[w], 2.0);  // 2/1
        const double E = (double)e[w];
        y[w] = fma(E, c[12], fma(E, c[11], f[w] * p[w]));
        if (kEnds) y[w] = x[w] < __builtin_huge_val() ? y[w] : x[w];
    }
}

// log x for normal positive x, +inf or NaN.
__device__ inline double det_log(double x)
{
    const double a[1] = {x};
    double y[1];
    det_log_w<1, true>(a, y);
    return y[0];
}

// atan z (any z).
__device__ inline double det_atan(double z)
{
    if (z != z) return z;
    const bool neg = z < 0.0;
    double a = neg ? -z : z;
    const bool inv = a > 1.0;
    if (inv) a = 1.0 / a;
    double r;
    if (a < 0x1p-800) {
        // both halvings are exact powers of two here (a^2 + 1 = 1), but the
        // general operators round a subnormal a / 2 as the definition does
        a = a / 2.0;
        a = a / 2.0;
        r = 4.0 * a;
    } else {
        const cdouble *c = coef_table(kAtanTab);
        double v[1] = {a}, t[1], u[1], s[1], p[1];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            t[0] = fma(v[0], v[0], 1.0);
            det_sqrt_w<1>(t, u);
            u[0] = 1.0 + u[0];
            det_div_w<1>(v, u, v);
        }
        s[0] = -(v[0] * v[0]);
        p[0] = c[0];
#pragma unroll
        for (int k = 1; k < 12; ++k) p[0] = fma_sc(p[0], s[0], c[k]);
        p[0] = fma(p[0], s[0], 1.0);
        r = 4.0 * (v[0] * p[0]);
    }
    if (inv) r = (0x1.921fb54442d18p+0 - r) + 0x1.1a62633145c07p-54;
    return neg ? -r : r;
}

// ------------------------------------------------------------- Philox4x32-10
struct Philox4 {
    uint32_t v[4];
};

__host__ __device__ inline Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        // one 32 x 32 -> 64-bit product per multiplier (a single v_mad_u64_u32)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t h0 = (uint32_t)(p0 >> 32), l0 = (uint32_t)p0;
        const uint32_t h1 = (uint32_t)(p1 >> 32), l1 = (uint32_t)p1;
        const uint32_t n0 = h1 ^ c1 ^ k0, n2 = h0 ^ c3 ^ k1;
        c0 = n0;
        c1 = l1;
        c2 = n2;
        c3 = l0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return Philox4{{c0, c1, c2, c3}};
}

// Random-number streams of the sampler.  Counter words: particle index,
// (pair << 16) | attempt, iteration, (stream tag << 24) | sampler id.
enum : uint32_t { kTagInit = 1, kTagPropose = 2, kTagResample = 3 };

__host__ __device__ inline Philox4 draw(uint64_t seed, uint32_t tag, uint32_t sampler, uint32_t t,
                                        uint32_t idx, uint32_t sub)
{
    return philox4x32_10(idx, sub, t, (tag << 24) | (sampler & 0xFFFFFFu), (uint32_t)seed,
                         (uint32_t)(seed >> 32));
}

__host__ __device__ inline uint64_t resample_word(uint64_t seed, uint32_t sampler, uint32_t t)
{
    const Philox4 w = draw(seed, kTagResample, sampler, t, 0u, 0u);
    return ((uint64_t)w.v[1] << 32) | w.v[0];
}

}  // namespace smc
