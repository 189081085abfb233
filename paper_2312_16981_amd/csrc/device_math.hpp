// Device-side scalar building blocks of the UGKWP hot path (gfx950).
//
//  - keyed counter-based random numbers: Philox4x32-10 (Salmon et al., SC'11);
//    the paper only requires eta ~ U(0,1) (Sec. 2.2, collision times;
//    Appendix A, frequencies);
//  - the group Planck integral behind B_g (Sec. 2.1);
//  - the UGKS time-averaged flux coefficients C4, C4 - e^{-s} (Sec. 2.2,
//    F^{fr,UGKS}, F^{fr,wave}) and C2 (Eq. C2Formula);
//  - the linear-frequency sampler (Eqs. Blinear, kg; Appendix A).
//
// Every expression that feeds a discrete decision (a collision test, a face
// crossing, a particle count) is written in a fixed evaluation order; the
// library is compiled with floating-point contraction off so the rounding is
// exactly that of the written order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ugk {

enum : uint32_t { PURPOSE_BIRTH = 1, PURPOSE_FLIGHT = 2 };

// pi^4 / 15 = int_0^inf t^3/(e^t-1) dt
#define UGK_PI4_15 6.49393940226682914909602217
#define UGK_15_PI4 0.153989733820265027837291749

struct Philox4 { uint32_t v[4]; };

// a ^ b ^ c; BITOP3: in one instruction.  (The 2-D push is slower for it, 750 us against
// 735 for 34 million particles; the 1-D push and the sampling faster, 31.0 against 31.3
// and 18.7 against 19.5 us for 1.3 million.)
template <bool BITOP3>
__host__ __device__ inline uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
#ifdef __HIP_DEVICE_COMPILE__
    if (BITOP3) return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#endif
    return a ^ b ^ c;
}

template <bool BITOP3 = true>
__host__ __device__ inline Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t lo = (uint64_t)0xD2511F53u * c0;
        const uint64_t hi = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3<BITOP3>((uint32_t)(hi >> 32), c1, k0);
        const uint32_t n2 = xor3<BITOP3>((uint32_t)(lo >> 32), c3, k1);
        c1 = (uint32_t)hi;
        c3 = (uint32_t)lo;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    Philox4 o;
    o.v[0] = c0; o.v[1] = c1; o.v[2] = c2; o.v[3] = c3;
    return o;
}

// Two 52-bit uniforms in (0,1) per Philox call: u = (k + 1/2) 2^-52.
__host__ __device__ inline double u52(uint32_t hi, uint32_t lo)
{
    const uint64_t k = ((uint64_t)hi << 20) | (uint64_t)(lo >> 12);
    return ((double)k + 0.5) * 2.220446049250313080847e-16;   // 2^-52
}

// Draw d of (seed, particle id, step, purpose): counter (id_lo, id_hi, step,
// purpose<<24 | d/2), key (seed_lo, seed_hi); even d takes words 0,1, odd d 2,3.
__host__ __device__ inline double keyed_uniform(uint64_t seed, uint64_t id, uint32_t step,
                                                uint32_t purpose, uint32_t d)
{
    const Philox4 r = philox4x32_10((uint32_t)id, (uint32_t)(id >> 32), step,
                                    (purpose << 24) | (d >> 1), (uint32_t)seed,
                                    (uint32_t)(seed >> 32));
    return (d & 1u) ? u52(r.v[2], r.v[3]) : u52(r.v[0], r.v[1]);
}

// Both draws of one Philox call (d0 even): out0 = draw d0, out1 = draw d0+1.
template <bool BITOP3 = true>
__host__ __device__ inline void keyed_uniform_pair(uint64_t seed, uint64_t id, uint32_t step,
                                                   uint32_t purpose, uint32_t d0, double& out0,
                                                   double& out1)
{
    const Philox4 r = philox4x32_10<BITOP3>((uint32_t)id, (uint32_t)(id >> 32), step,
                                    (purpose << 24) | (d0 >> 1), (uint32_t)seed,
                                    (uint32_t)(seed >> 32));
    out0 = u52(r.v[0], r.v[1]);
    out1 = u52(r.v[2], r.v[3]);
}

// ---------------------------------------------------------------------------
// Polynomial coefficients of the functions below, interpolated in 60-digit
// arithmetic at the Chebyshev nodes of each interval (gen_math_tab.py), in ascending
// order.  They are read from constant memory with scalar loads (math_tab) and enter each
// multiply-add as a scalar operand (horner): as literals every one of them cost two
// vector moves beside its multiply-add, 40% of a source-iteration sweep's vector
// instructions.
struct MathTab {
    double head[11], weight[11], L1[11], L2[10], L3[10], L4[9];   // Planck edge integrals
    double ex[10];        // (e^{-r} - 1 + r) / r^2 on |r| <= ln 2 / 2
    double exf[11];       // the same within 5e-18
    double one_ex[15];    // (1 - e^{-x}) / x on [0, 2]
    double w[12];         // (C4 - e^{-s}) / s on [0, 1]
    double c2[15];        // (C2/dt) / s on [0, 2]
    double ln[7];         // (atanh(s) / s - 1) / z of z = s^2 on [0, 0.02944]
};

static __device__ __constant__ MathTab g_math_tab = {
    // head
    {
        0x1.1111111111111p-6, -0x1.a01a01a01a00cp-13, 0x1.ed284dc73913ap-19,
        -0x1.42cb40de6ce69p-24, 0x1.b96d78ff346dfp-30, -0x1.35de2d321efc1p-35,
        0x1.bb24e628870e6p-41, -0x1.4129968cff7fdp-46, 0x1.d2ff446f590b8p-52,
        -0x1.4167e3777db0cp-57, 0x1.3c38f7b6766edp-63},
    // weight
    {
        0x1.5555555555555p-4, -0x1.6c16c16c16be9p-10, 0x1.1566abc00dc60p-15,
        -0x1.bbd7792fd1d51p-21, 0x1.66a8f1dec7df9p-26, -0x1.22803c5468dd9p-31,
        0x1.d6d514ef48785p-37, -0x1.7d480a243cf13p-42, 0x1.31c14b6cc26a3p-47,
        -0x1.c85ef977724aep-53, 0x1.db16cc9ec36f6p-59},
    // L1, L2, L3, L4
    {
        0x1.0000000000000p-1, 0x1.55555555552abp-2, 0x1.0000000031175p-2,
        0x1.9999996d9bf5ep-3, 0x1.55555f69ddceep-3, 0x1.2490f16d2c5aap-3,
        0x1.001c65f48b967p-3, 0x1.c41ed2a88b55ap-4, 0x1.b32a2f68f50a9p-4,
        0x1.e02d976230df8p-5, 0x1.5fe2649cd3a3bp-3},
    {
        0x1.ffffffffffffep-3, 0x1.c71c71c71dbeap-4, 0x1.fffffffd87c9cp-5,
        0x1.47ae156328546p-5, 0x1.c71c1b62233dap-6, 0x1.4e673a88c4a0ep-6,
        0x1.fed17383d92dep-7, 0x1.a073e8eee8b18p-7, 0x1.00b994566244cp-7,
        0x1.ec3cb78ada50ap-7},
    {
        0x1.0000000000000p-3, 0x1.2f684bda132b7p-5, 0x1.ffffffff37066p-7,
        0x1.0624dd78f9432p-7, 0x1.2f68305bc51abp-8, 0x1.7e282f8ebf2f2p-9,
        0x1.ff3ef85d092edp-10, 0x1.6f35ac8fe074fp-10, 0x1.b130dc87cf843p-11,
        0x1.543bfa02e9c77p-10},
    {
        0x1.0000000000001p-4, 0x1.948b0fcd6c85bp-7, 0x1.0000000337272p-8,
        0x1.a36e2ae7b4a04p-10, 0x1.948c2d1b9aa6ap-11, 0x1.b48aa20035ed0p-12,
        0x1.023e6d3996791p-12, 0x1.2022a1c4b980ep-13, 0x1.4405e264f325cp-13},
    // ex
    {
        0x1.0000000000001p-1, -0x1.5555555555556p-3, 0x1.5555555553d63p-5, -0x1.11111111109b3p-7, 0x1.6c16c1788bd90p-10,
        -0x1.a01a01a7c41d5p-13, 0x1.a019b90d2ae7ap-16, -0x1.71de0dae63bb3p-19, 0x1.289185613a3d6p-22,
        -0x1.af38a9b0ec855p-26},
    // exf
    {
        0x1.0000000000000p-1, -0x1.5555555555557p-3, 0x1.5555555555556p-5, -0x1.11111111100dcp-7, 0x1.6c16c16c162d4p-10,
        -0x1.a01a01abe7fe1p-13, 0x1.a01a01a6d889cp-16, -0x1.71de0231960ebp-19, 0x1.27e4db646b17ep-22,
        -0x1.af4de97ca4194p-26, 0x1.1f730349868cep-29},
    // one_ex
    {
        0x1.0000000000000p+0, -0x1.ffffffffffffbp-2, 0x1.55555555553e2p-3, -0x1.555555554ff99p-5, 0x1.111111106b15bp-7,
        -0x1.6c16c153ded1bp-10, 0x1.a019ff50cb17dp-13, -0x1.a019dae22ccbcp-16, 0x1.71dc6e07bfee1p-19,
        -0x1.27d5968445595p-22, 0x1.ada5400e8ee01p-26, -0x1.1b960644cf556p-29, 0x1.4bed628f79b85p-33,
        -0x1.375240aee064dp-37, 0x1.566ca7300ffc9p-42},
    // w
    {
        0x1.0000000000000p-1, -0x1.5555555555519p-2, 0x1.fffffffffd314p-4, -0x1.11111110a7febp-5, 0x1.c71c71a754d26p-8,
        -0x1.38137e610a937p-10, 0x1.6c166edfaf704p-13, -0x1.71d809f19c654p-16, 0x1.4c91f8a6b2e53p-19,
        -0x1.0a541db8a7dfdp-22, 0x1.6d0ad6972752dp-26, -0x1.4e8a878a9e670p-30},
    // c2
    {
        -0x1.5555555555555p-3, 0x1.5555555555554p-4, -0x1.99999999998f7p-6,
        0x1.6c16c16c146a9p-8, -0x1.04104103c7cf0p-10, 0x1.3813812d8237ep-13,
        -0x1.43a27208d508ap-16, 0x1.27e4ea93c9d63p-19, -0x1.e42f503d5530dp-23,
        0x1.669b8c12ac8e5p-26, -0x1.e4ebe34da03a0p-30, 0x1.2bcb054dfb2d6p-33,
        -0x1.4b6b8af1e10c9p-37, 0x1.29366afc1960cp-41, -0x1.3d06be2fd103fp-46},
    // ln
    {
        0x1.5555555555558p-2, 0x1.99999999952e2p-3, 0x1.2492492df1492p-3,
        0x1.c71c62e57fa3fp-4, 0x1.7462b4ab4c062p-4, 0x1.39fe60617ce73p-4,
        0x1.2b584add1c619p-4}
};

#ifdef __HIP_DEVICE_COMPILE__
typedef const __attribute__((address_space(4))) MathTab* TabPtr;
typedef const __attribute__((address_space(4))) double* CoefPtr;
#else
typedef const MathTab* TabPtr;
typedef const double* CoefPtr;
#endif

// The table, by an address the compiler does not know: a loop that asks for it
// in its body loads the coefficients there instead of keeping all of them in
// registers throughout.
__device__ inline TabPtr math_tab()
{
    TabPtr p = (TabPtr)&g_math_tab;
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+s"(p));
#endif
    return p;
}

// Horner steps a = a x + c with the coefficients in scalar registers: the compiler
// prefers the two-operand multiply-add, whose addend is also its destination, and
// copies each coefficient to vector registers first.  The s_nop covers the two wait
// states between a vector instruction that writes a scalar register (a spilled
// coefficient read back from a lane) and its use here, which the compiler counts only
// for instructions it knows; callers likewise pass the result through an operation of
// their own before any cross-lane move.
#ifdef __HIP_DEVICE_COMPILE__
#define UGK_FMA "v_fma_f64 %0, %0, %1, "
#endif
template <int N>
__device__ inline double horner(CoefPtr c, double a, double x)
{
#ifdef __HIP_DEVICE_COMPILE__
    if constexpr (N >= 4) {
        asm("s_nop 1\n\t" UGK_FMA "%2\n\t" UGK_FMA "%3\n\t" UGK_FMA "%4\n\t" UGK_FMA "%5"
            : "+&v"(a) : "v"(x), "s"(c[N - 1]), "s"(c[N - 2]), "s"(c[N - 3]), "s"(c[N - 4]));
        return horner<N - 4>(c, a, x);
    } else if constexpr (N == 3) {
        asm("s_nop 1\n\t" UGK_FMA "%2\n\t" UGK_FMA "%3\n\t" UGK_FMA "%4"
            : "+&v"(a) : "v"(x), "s"(c[2]), "s"(c[1]), "s"(c[0]));
    } else if constexpr (N == 2) {
        asm("s_nop 1\n\t" UGK_FMA "%2\n\t" UGK_FMA "%3" : "+&v"(a) : "v"(x), "s"(c[1]), "s"(c[0]));
    } else if constexpr (N == 1) {
        asm("s_nop 1\n\t" UGK_FMA "%2" : "+&v"(a) : "v"(x), "s"(c[0]));
    }
    return a;
#else
    for (int j = N - 1; j >= 0; --j) a = fma(a, x, c[j]);
    return a;
#endif
}

// c[0] + x (c[1] + ... + x c[N-1])
#ifdef __HIP_DEVICE_COMPILE__
template <int N>
__device__ inline double poly(const __attribute__((address_space(4))) double (&c)[N], double x)
{
    return horner<N - 2>((CoefPtr)&c[0], fma(x, c[N - 1], c[N - 2]), x);
}
#endif

template <int N>
__device__ inline double poly(const double (&c)[N], double x)
{
    double acc = c[N - 1];
#pragma unroll
    for (int j = N - 2; j >= 0; --j) acc = fma(acc, x, c[j]);
    return acc;
}

// -ln(u) for u in (0, 1), the uniforms above.  u = 2^e m with m in
// [sqrt(1/2), sqrt(2)); ln m = 2 atanh(s) with s = (m - 1)/(m + 1), |s| <= 0.1716,
// as 2s (1 + z q(z)), z = s^2, q of degree 6 (z q within 5e-18).  ln 2 is split so that
// e ln2_hi is exact (ln2_hi keeps 32 significant bits).  The result is within a few ulp
// of the correctly rounded value; the tests compare it with the host libm.
// LITERAL: the coefficients in the code rather than in the table (the 2-D push: 735 us
// against 755 with the scalar loads; the 1-D push's registers fall from 95 to 83 with them).
template <bool LITERAL = false>
__device__ inline double neg_log_unit(double u)
{
    int e;
    double m = frexp(u, &e);                       // u = m 2^e, m in [1/2, 1)
    if (m < 0.70710678118654752440) {
        m = m + m;
        e -= 1;
    }
    const double s = (m - 1.0) / (m + 1.0);        // m - 1 is exact here
    const double z = s * s, t = s + s;
    double q;
    if (LITERAL) {
        q = 0x1.2b584add1c619p-4;
        q = fma(q, z, 0x1.39fe60617ce73p-4);
        q = fma(q, z, 0x1.7462b4ab4c062p-4);
        q = fma(q, z, 0x1.c71c62e57fa3fp-4);
        q = fma(q, z, 0x1.2492492df1492p-3);
        q = fma(q, z, 0x1.99999999952e2p-3);
        q = fma(q, z, 0x1.5555555555558p-2);
    } else {
        q = poly<7>(math_tab()->ln, z);
    }
    const double lnm = fma(t, z * q, t);
    const double de = (double)e;
    const double ln2_hi = 0x1.62e42fee00000p-1, ln2_lo = 0x1.a39ef35793c76p-33;
    return -fma(de, ln2_hi, fma(de, ln2_lo, lnm));
}

// The coefficients of the Planck integrals and the exponential kept in vector
// registers: for blocks too few to hide the scalar loads' latency behind each other.
struct RegTab {
    double head[11], weight[11], L1[11], L2[10], L3[10], L4[9], ex[10];
    __device__ inline const RegTab* operator->() const { return this; }
};

// W: with the edge weights' coefficients.
template <bool W>
__device__ inline RegTab reg_tab()
{
    const TabPtr t = math_tab();
    RegTab r;
#ifdef __HIP_DEVICE_COMPILE__
#define UGK_KEEP(x) asm volatile("" : "+v"(x))
#else
#define UGK_KEEP(x)
#endif
#pragma unroll
    for (int j = 0; j < 11; ++j) {
        r.head[j] = t->head[j];
        r.L1[j] = t->L1[j];
        r.weight[j] = W ? t->weight[j] : 0.0;
        UGK_KEEP(r.head[j]);
        UGK_KEEP(r.L1[j]);
        if (W) UGK_KEEP(r.weight[j]);
    }
#pragma unroll
    for (int j = 0; j < 10; ++j) {
        r.L2[j] = t->L2[j];
        r.L3[j] = t->L3[j];
        r.ex[j] = t->ex[j];
        UGK_KEEP(r.L2[j]);
        UGK_KEEP(r.L3[j]);
        UGK_KEEP(r.ex[j]);
    }
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        r.L4[j] = t->L4[j];
        UGK_KEEP(r.L4[j]);
    }
#undef UGK_KEEP
    return r;
}

// e^{-x} for any x (inf for NaN): x = k ln 2 + r with |r| <= ln 2 / 2 (ln 2
// in two parts, k times the first exact), e^{-r} = 1 - r + r^2 q(r), q of degree 9 within 2e-16.
template <class Tab>
__device__ inline double exp_neg(const Tab& t, double x)
{
    x = fmin(fmax(x, -800.0), 800.0);
    const double k = rint(x * 0x1.71547652b82fep+0);
    const double r = fma(-k, 0x1.473de6af278edp-34, fma(-k, 0x1.62e42fef00000p-1, x));
    const double p = fma(r, fma(r, poly<10>(t->ex, r), -1.0), 1.0);
    return ldexp(p, -(int)k);
}

// e^{-x} in two parts, 2^-k (hi + lo): with the rounding errors of r and of 1 - r, and q of
// degree 10 (within 5e-18).
struct ExpParts {
    double hi, lo;
    int k;
};

__device__ inline ExpParts exp_parts(TabPtr t, double x)
{
    x = fmin(fmax(x, -800.0), 800.0);
    const double k = rint(x * 0x1.71547652b82fep+0), a = fma(-k, 0x1.62e42fef00000p-1, x);
    const double r = fma(-k, 0x1.473de6af278edp-34, a), dr = fma(-k, 0x1.473de6af278edp-34, a - r);
    const double h = 1.0 - r, l = fma(r * r, poly<11>(t->exf, r), ((1.0 - h) - r) - dr), hi = h + l;
    return {hi, l - (hi - h), (int)k};
}

// e^{-x} where its own rounding is the result's: 1.11e-16 at most, as libm's (exp_neg: 1.43e-16).
__device__ inline double exp_neg_fine(TabPtr t, double x)
{
    const ExpParts e = exp_parts(t, x);
    return ldexp(e.hi, -e.k);
}

// 1 - e^{-x} for x >= 0: within 1.41e-16, as expm1.
__device__ inline double one_less_exp_neg(TabPtr t, double x)
{
    const ExpParts e = exp_parts(t, x);
    const double hi = ldexp(e.hi, -e.k), w = 1.0 - hi;
    return w + (((1.0 - w) - hi) - ldexp(e.lo, -e.k));
}

// n / d with r = 1/d at hand: one correction of n r (the quotient to the last
// bit but for rare half-way cases), 3 instructions instead of a division's 11.
__host__ __device__ inline double quotient(double n, double d, double r)
{
    const double q = n * r;
    return fma(fma(-d, q, n), r, q);
}

// v / 6 (Simpson's rule) and v / (pi^4 / 15)
__host__ __device__ inline double sixth(double v) { return quotient(v, 6.0, 1.0 / 6.0); }
__host__ __device__ inline double over_pi4_15(double v) { return quotient(v, UGK_PI4_15, UGK_15_PI4); }

// ---------------------------------------------------------------------------
// Planck band integrals.  head(x) = int_0^x t^3/(e^t-1) dt below x = 2,
// tail(x) = int_x^inf t^3/(e^t-1) dt = sum_n e^{-nx}(x^3/n + 3x^2/n^2 + 6x/n^3 + 6/n^4) from 2 on.
//
// Both are evaluated with polynomials of fixed degree:
//  - head = x^3 (1/3 - x/8 + x^2 q(x^2)), q of degree 10 on x^2 < 4 (the Bernoulli
//    series of the integrand; error 4e-19 of q);
//  - with z = e^{-x} <= e^{-2}, tail = z (x^3 + 3x^2 + 6x + 6) +
//    z^2 (x^3 L1(z) + 3x^2 L2(z) + 6x L3(z) + 6 L4(z)), L_m = sum_{n>=2} z^{n-2} / n^m of
//    degrees 10, 9, 9, 8: the z^2 part is at most 3% of the value and each L_m is within
//    5e-17 of its series, so that the rounding of the first part is what is left;
//  - the edge weight x^4/(e^x-1) = x head'(x) from the Bernoulli series below 2 and
//    x^4 z/(1-z) above, where nothing cancels.
// A fixed count of multiply-adds (four short chains for the tail) replaces a
// series of up to 60 terms that ran until its slowest lane was done: the
// sweeps are bound by their double-precision instructions, and a wavefront
// holds both sides of x = 2.  Tab: TabPtr or RegTab.
template <class Tab>
__device__ inline double planck_head(const Tab& t, double x)
{
    const double x2 = x * x;
    return x2 * x * fma(x2, poly<11>(t->head, x2), fma(x, -0.125, 1.0 / 3.0));
}

// z = e^{-x} > 0
template <class Tab>
__device__ inline double planck_tail(const Tab& t, double x, double z)
{
    const double p1 = fma(fma(x + 3.0, x, 6.0), x, 6.0);
    const double hi = fma(fma(poly<11>(t->L1, z), x, 3.0 * poly<10>(t->L2, z)), x, 6.0 * poly<10>(t->L3, z));
    return z * fma(z, fma(hi, x, 6.0 * poly<9>(t->L4, z)), p1);
}

template <class Tab>
__device__ inline double planck_weight_head(const Tab& t, double x)
{
    const double x2 = x * x;
    return x2 * x * fma(x2, poly<11>(t->weight, x2), fma(x, -0.5, 1.0));
}

// Edge value used by group bands: head(x) below 2, tail(x) from 2 on.
template <class Tab>
__device__ inline double planck_edge_value(const Tab& t, double x)
{
    if (x < 2.0) return planck_head(t, x);
    const double z = exp_neg(t, x);
    return z == 0.0 ? 0.0 : planck_tail(t, x, z);
}

// x^4 / (e^x - 1): the edge term of d phi_g / dT (the band integral of a
// group differentiated through its limits nu / T)
template <class Tab>
__device__ inline double planck_edge_weight(const Tab& t, double x)
{
    if (x < 2.0) return planck_weight_head(t, x);
    const double z = exp_neg(t, x), x2 = x * x;
    return z == 0.0 ? 0.0 : x2 * x2 * (z / (1.0 - z));
}

// Both, with one exponential.
template <class Tab>
__device__ inline void planck_edge_both(const Tab& t, double x, double* v, double* w)
{
    if (x < 2.0) {
        *v = planck_head(t, x);
        *w = planck_weight_head(t, x);
        return;
    }
    const double z = exp_neg(t, x), x2 = x * x;
    *v = z == 0.0 ? 0.0 : planck_tail(t, x, z);
    *w = z == 0.0 ? 0.0 : x2 * x2 * (z / (1.0 - z));
}

// int_{xl}^{xh} t^3/(e^t-1) from edge values vl = edge_value(xl), vh = edge_value(xh).
__device__ inline double planck_band_from_edges(double xl, double vl, double xh, double vh)
{
    if (xh < 2.0) return vh - vl;                       // both heads
    if (xl < 2.0) return (UGK_PI4_15 - vl) - vh;        // head below, tail above
    return vl - vh;                                     // both tails
}

// phi_g(T) = a c T^4 (15/pi^4) band
__device__ inline double phi_from_band(double a, double c, double T, double band)
{
    const double T2 = T * T;
    return a * c * T2 * T2 * over_pi4_15(band);
}

// ---------------------------------------------------------------------------
// Flux coefficients as functions of s = c sigma dt / eps^2.

__device__ inline double coef_c4(TabPtr t, double s)
{
    return s < 2.0 ? poly<15>(t->one_ex, s) : (1.0 - exp_neg(t, s)) / s;
}

// The power-series coefficients of the functions below, fixed at compile time
// (each a ratio of integers rounded once), so that a term costs a multiply
// and no division.  Index n is the series' own summation index.
struct SeriesCoefs {
    double c5[81];    // 1 / (n! (n+2))                   C5/dt
    double w5[81];    // n / (2 n! (n+2))                 (C5 + dt/2 e^{-s})/dt
    double wos[61];   // n / (n+1)!                       (C4 - e^{-s})/s
    double c2ds[81];  // (n-1)^2 / (n+1)!                 d(C2/dt)/ds
};

constexpr SeriesCoefs make_series_coefs()
{
    SeriesCoefs t{};
    double fact = 1.0;                       // n!
    for (int n = 0; n < 81; ++n) {
        if (n > 0) fact *= (double)n;
        const double fact1 = fact * (double)(n + 1);     // (n+1)!
        if (n < 61) t.wos[n] = (double)n / fact1;
        t.c5[n] = 1.0 / (fact * (double)(n + 2));
        t.w5[n] = (double)n / (2.0 * fact * (double)(n + 2));
        t.c2ds[n] = (double)((n - 1) * (n - 1)) / fact1;
    }
    return t;
}

constexpr SeriesCoefs kSeries = make_series_coefs();

// C4 - e^{-s}: below s = 1, where that cancels, s times the polynomial of its series
// sum_{n>=1} (-1)^{n+1} n s^n/(n+1)! (within 4e-17).
__device__ inline double coef_w(TabPtr t, double s)
{
    return s < 1.0 ? s * poly<12>(t->w, s) : coef_c4(t, s) - exp_neg(t, s);
}

// C2/dt = [2 C4 - 1 - e^{-s}] / s from s = 2 on; below, where that cancels, s times the
// polynomial of the series sum_{n>=2} (-1)^{n+1} (n-1) s^{n-1}/(n+1)! (within 1e-18).
// (1/s is 0 for an infinite s alone, whose quotients would be NaN.)
__device__ inline double coef_c2_over_dt(TabPtr t, double s)
{
    if (s < 2.0) return s * poly<15>(t->c2, s);
    const double e = exp_neg(t, s), r = 1.0 / s;
    const double c4 = quotient(1.0 - e, s, r);
    return r > 0.0 ? quotient(2.0 * c4 - 1.0 - e, s, r) : -r;
}

// C5/dt of the slope term of the UGKS free-transport flux (Sec. 2.2):
// -int_0^1 u e^{-s u} du = ((1 + s) e^{-s} - 1) / s^2.  Below s = 2 the
// expansion -1/2 + s/3 - s^2/8 + ... = sum_n (-1)^{n+1} s^n / (n! (n+2)).
__host__ __device__ inline double coef_c5(double s)
{
    if (s < 2.0) {
        double p = 1.0, sum = -0.5;                      // n = 0 term
        for (int n = 1; n < 80; ++n) {
            p *= s;
            const double t = kSeries.c5[n] * p;
            sum += (n & 1) ? t : -t;
            if (t < 1e-18 * fabs(sum)) break;
        }
        return sum;
    }
    return ((1.0 + s) * exp(-s) - 1.0) / (s * s);
}

// (C5 + (dt/2) e^{-s}) / dt, the slope coefficient of the wave flux of a
// sampled cell; below s = 2, sum_{n>=1} (-1)^n n s^n / (2 n! (n+2)) (the two
// terms of the closed form cancel as s -> 0).
__host__ __device__ inline double coef_w5(double s)
{
    if (s < 2.0) {
        double p = 1.0, sum = 0.0;
        for (int n = 1; n < 80; ++n) {
            p *= s;
            const double t = kSeries.w5[n] * p;
            sum += (n & 1) ? -t : t;
            if (t < 1e-18 * fabs(sum)) break;
        }
        return sum;
    }
    return coef_c5(s) + 0.5 * exp(-s);
}

// Derivatives in s (for the adjoint of the macroscopic solve).  With
// W/s -> 1/2 as s -> 0 taken from W's series below s = 1:
//   C4' = -W/s,   W' = e^{-s} - W/s,   (C2/dt)' = (e^{-s} - 2 W/s - C2/dt) / s,
// the last replaced below s = 2 by its series
//   sum_{n>=2} (-1)^{n+1} (n-1)^2 s^{n-2} / (n+1)!   (it cancels there).
__host__ __device__ inline double coef_w_over_s(double s)
{
    if (s < 1.0) {
        double p = 1.0, sum = 0.5;                      // n = 1 term: 1/2
        for (int n = 2; n < 60; ++n) {
            p *= s;                                     // s^{n-1}
            const double t = kSeries.wos[n] * p;
            sum += (n & 1) ? t : -t;
            if (t < 1e-18 * fabs(sum)) break;
        }
        return sum;
    }
    return (-expm1(-s) / s - exp(-s)) / s;
}

__host__ __device__ inline double coef_c4_ds(double s) { return -coef_w_over_s(s); }

__host__ __device__ inline double coef_w_ds(double s) { return exp(-s) - coef_w_over_s(s); }

__device__ inline double coef_c2_over_dt_ds(TabPtr t, double s)
{
    if (s < 2.0) {
        double p = 1.0, sum = -1.0 / 6.0;               // n = 2 term
        for (int n = 3; n < 80; ++n) {
            p *= s;                                     // s^{n-2}
            const double q = kSeries.c2ds[n] * p;
            sum += (n & 1) ? q : -q;
            if (q < 1e-18 * fabs(sum)) break;
        }
        return sum;
    }
    return (exp(-s) - 2.0 * coef_w_over_s(s) - coef_c2_over_dt(t, s)) / s;
}

// ---------------------------------------------------------------------------
// Linear-frequency sampling.  beta = (B(nh) - B(nl)) / B(nmid) limited to [-2, 2]
// (keeps the linear pdf non-negative on the group); evaluated as ratios of
// Planck functions so that nothing under- or overflows for steep Wien tails.
__host__ __device__ inline double freq_slope(double nl, double nh, double T)
{
    const double nm = 0.5 * (nl + nh);
    const double em = -expm1(-nm / T);
    const double rh = nh / nm, rl = nl / nm;
    const double bh = rh * rh * rh * exp(-(nh - nm) / T) * em / (-expm1(-nh / T));
    const double bl = rl * rl * rl * exp(-(nl - nm) / T) * em / (-expm1(-nl / T));
    double beta = bh - bl;
    beta = beta > 2.0 ? 2.0 : beta;
    beta = beta < -2.0 ? -2.0 : beta;
    return beta;
}

// Inverse CDF of the pdf (1 + beta u')/dnu, u' = (nu - nmid)/dnu in [-1/2, 1/2]:
// (beta/2) u'^2 + u' + q = 0, q = 1/2 - beta/8 - U, stable root -2q/(1 + sqrt(1 - 2 beta q)).
__host__ __device__ inline double sample_nu(double nl, double nh, double beta, double U)
{
    const double nm = 0.5 * (nl + nh);
    const double dnu = nh - nl;
    const double q = 0.5 - 0.125 * beta - U;
    double disc = 1.0 - 2.0 * beta * q;
    disc = disc < 0.0 ? 0.0 : disc;
    const double up = -2.0 * q / (1.0 + sqrt(disc));
    double nu = nm + up * dnu;
    nu = nu < nl ? nl : nu;
    nu = nu > nh ? nh : nu;
    return nu;
}

// Offset u' in [-1/2, 1/2] whose CDF under the density 1 + beta u' is U
// (the same quadratic as sample_nu); places new particles along the slope of
// their cell's wave part.
__host__ __device__ inline double linear_offset(double beta, double U)
{
    const double q = 0.5 - 0.125 * beta - U;
    double disc = 1.0 - 2.0 * beta * q;
    disc = disc < 0.0 ? 0.0 : disc;
    return -2.0 * q / (1.0 + sqrt(disc));
}

// ---------------------------------------------------------------------------
// Olson's material (Sec. 3.4, Eq. cvolson).  The ionisation fraction alpha solves
// alpha^2 = e^{-chi/T} (1 - alpha); with h = e^{-chi/(2T)} and r = sqrt(h^2 + 4) it is
// h (r - h)/2 (no overflow for cold material), and dalpha/dT = (chi/T^2)(alpha - h/r).
__host__ __device__ inline double olson_alpha(double T, double chi, double* dalpha)
{
    const double h = exp(-0.5 * chi / T);
    const double r = sqrt(h * h + 4.0);
    const double al = 0.5 * h * (r - h);
    if (dalpha) *dalpha = (chi / (T * T)) * (al - h / r);
    return al;
}

// Heat capacity H [1 + alpha + (T + chi) alpha'] (the printed a T_keV^3 is the unit
// a (1 keV)^3, folded into H) and the material energy H [T (1 + alpha) + chi alpha]
// whose derivative it is.
__host__ __device__ inline double olson_cv(double H, double chi, double T)
{
    double da;
    const double al = olson_alpha(T, chi, &da);
    return H * (1.0 + al + (T + chi) * da);
}

__host__ __device__ inline double olson_energy(double H, double chi, double T)
{
    const double al = olson_alpha(T, chi, nullptr);
    return H * (T * (1.0 + al) + chi * al);
}

// The temperature whose Olson material energy is u > 0.  The energy rises
// strictly with T: a bracket [lo, hi] with energy(lo) <= u <= energy(hi) is found
// by doubling from T0, then Newton steps from T0 that stay inside the bracket
// (else its midpoint), until a step moves T by at most 1e-15 T.  Returns -1 for
// u <= 0 (no temperature).
__host__ __device__ inline double olson_temperature(double H, double chi, double u, double T0)
{
    if (!(u > 0.0) || !isfinite(u)) return -1.0;
    double lo = 0.0, hi = T0 > 0.0 ? T0 : 1.0;
    for (int n = 0; n < 2100 && olson_energy(H, chi, hi) < u; ++n) {
        lo = hi;
        hi = 2.0 * hi;
    }
    double T = (T0 > lo && T0 < hi) ? T0 : 0.5 * (lo + hi);
    for (int n = 0; n < 200; ++n) {
        const double f = olson_energy(H, chi, T) - u;
        if (f == 0.0) break;
        if (f < 0.0) lo = T; else hi = T;
        double Tn = T - f / olson_cv(H, chi, T);
        if (!(Tn > lo && Tn < hi)) Tn = 0.5 * (lo + hi);
        const double d = fabs(Tn - T);
        T = Tn;
        if (d <= 1e-15 * T) break;
    }
    return T;
}

// ---------------------------------------------------------------------------
// Tabulated opacity: the interval [i, i+1] of n ascending nodes holding x and the
// weight of node i+1 (clamped to the end intervals: weight 0 or 1 beyond them).
__host__ __device__ inline int table_locate(const double* nodes, int n, double x, double* frac)
{
    if (x <= nodes[0]) { *frac = 0.0; return 0; }
    if (x >= nodes[n - 1]) { *frac = 1.0; return n - 2; }
    int lo = 0, hi = n - 1;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (nodes[mid] <= x) lo = mid; else hi = mid;
    }
    *frac = (x - nodes[lo]) / (nodes[lo + 1] - nodes[lo]);
    return lo;
}

// The same interval found from a first guess: for nodes evenly spaced from
// nodes[0] with 1/spacing inv (inv = 0: no guess, plain bisection) the guess is
// the interval of x on that grid, then moved until nodes[i] <= x < nodes[i+1]
// holds as bisection would leave it.  Same result as table_locate.
__host__ __device__ inline int table_locate_guess(const double* nodes, int n, double x, double inv,
                                                  double* frac)
{
    if (!(inv > 0.0)) return table_locate(nodes, n, x, frac);
    if (x <= nodes[0]) { *frac = 0.0; return 0; }
    if (x >= nodes[n - 1]) { *frac = 1.0; return n - 2; }
    double gq = (x - nodes[0]) * inv;
    int i = gq < 0.0 ? 0 : (gq > (double)(n - 2) ? n - 2 : (int)gq);
    while (i > 0 && nodes[i] > x) --i;
    while (i < n - 2 && nodes[i + 1] <= x) ++i;
    *frac = (x - nodes[i]) / (nodes[i + 1] - nodes[i]);
    return i;
}

// nu^-p with the exact cube for the paper's p = 3.
__host__ __device__ inline double nu_pow(double nu, double p)
{
    return p == 3.0 ? 1.0 / (nu * nu * nu) : pow(nu, -p);
}

}  // namespace ugk
