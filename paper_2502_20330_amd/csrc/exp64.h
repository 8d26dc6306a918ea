// fp64 exponentials of the accept pass (to be included after hip_runtime.h).
#pragma once

namespace {

constexpr double kLn2 = 0.6931471805599453;

// a * b + k with the constant in scalar registers: left to itself the compiler keeps each coefficient in a vector register
// pair (or copies it into one before every multiply-add), and the fifty of them spill the entries' own state.
__device__ __forceinline__ double fma_k(double a, double b, double k)
{
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(k));
    return d;
}
// Compact fp64 exponential (about twenty instructions, inlined where used): exp(x) with ~2e-16
// relative error for x <= 700; anything below -745 (also -inf and NaN) gives 0.  The decisions
// need fp64 but each workgroup runs its code exactly once, so instruction count matters more
// here than in a loop: the library routine is several times longer.
__device__ __forceinline__ double exp_c(double x)
{
    x = fmax(x, -746.0);
    const double k = rint(x * 1.4426950408889634);
    double r = fma(k, -6.93147180369123816490e-01, x);        // k ln2 in two parts (the split of fdlibm's e_exp.c)
    r = fma(k, -1.90821492927058770002e-10, r);
    double p = 1.0 / 6227020800.0;                           // Taylor to r^13 / 13!, |r| <= 0.347
    p = fma(p, r, 1.0 / 479001600.0);
    p = fma(p, r, 1.0 / 39916800.0);
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)k);
}
// The exponentials of accept_draw_row, millions of them at large batches: exp(x) = 2^e 2^(j/64) exp(r) with the
// powers in a table that the workgroup keeps in LDS, |r| <= ln2/128 and a polynomial of degree 5 whose coefficients also
// stand for the next term (Chebyshev economisation; Taylor's own would leave 4e-17).
// About two thirds of exp_c's time and as exact (at most 1.2e-16 relative error, exp_c 1.4e-16): the table also
// holds what rounding took from each power, without which it would be 2.3e-16 (a table of its own: pairs of doubles in one
// 128-bit read spilled registers).  Rounding to a multiple of ln2/64 by adding 1.5 2^52
// leaves the integer in the low word, which holds it up to 2^31 only: arguments are clamped above too, where the result
// is +inf already (a shift eta (q - p) may be of any size; without the clamp 2.4e7 gave 0).
struct Exp2 { double v[64]; float rest[64]; };      // 2^(j/64) = v (1 + rest)
__device__ const Exp2 kExp2Table = {
    {0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
     0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
     0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
     0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
     0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
     0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
     0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
     0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
     0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
     0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
     0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
     0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
     0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
     0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
     0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
     0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0},
    {0x0.0p+0f, -0x1.16013ap-56f, 0x1.cd2524p-55f, 0x1.0f74e6p-57f,
     0x1.79aa66p-54f, 0x1.ebe3d8p-60f, -0x1.556522p-54f, -0x1.1c923cp-54f,
     -0x1.01b15ep-55f, 0x1.b898c4p-55f, 0x1.aecf74p-54f, 0x1.a6f414p-55f,
     0x1.68efdep-54f, 0x1.0472bap-55f, 0x1.2f7e16p-55f, 0x1.b37828p-55f,
     0x1.34d754p-55f, 0x1.fdd396p-55f, -0x1.24aedcp-54f, -0x1.1d1e84p-56f,
     0x1.59f48ap-55f, -0x1.8a78f4p-58f, 0x1.363ed6p-59f, 0x1.ecce1ep-57f,
     0x1.690cecp-56f, -0x1.f94340p-55f, -0x1.8dec6cp-56f, 0x1.335052p-54f,
     0x1.063e1ep-54f, 0x1.432e62p-54f, -0x1.c33c54p-55f, -0x1.3cedd8p-54f,
     -0x1.3b3efcp-54f, -0x1.367efcp-57f, -0x1.81f648p-56f, -0x1.619322p-55f,
     -0x1.b32dccp-56f, 0x1.5ebe1ap-57f, -0x1.369b70p-54f, -0x1.4d450ep-54f,
     0x1.db72fcp-55f, 0x1.bf6836p-56f, -0x1.da9b88p-58f, -0x1.243432p-54f,
     0x1.1affc2p-56f, -0x1.7c5042p-55f, -0x1.1bbd1ep-54f, 0x1.469846p-55f,
     0x1.c1a77ap-55f, -0x1.5c3d96p-58f, -0x1.8d6f44p-57f, 0x1.4ffd70p-56f,
     0x1.36eae4p-56f, 0x1.4e08fep-55f, 0x1.76b2c6p-57f, -0x1.fad5d4p-55f,
     0x1.4a385ap-56f, 0x1.e5a50ep-55f, -0x1.2d5210p-55f, 0x1.4b6046p-56f,
     -0x1.ff7128p-55f, 0x1.ec3bc4p-55f, 0x1.a64a94p-55f, 0x1.7893b4p-56f}};
__device__ __forceinline__ double exp_tab(double x, const Exp2& tab)
{
    constexpr double kShift = 6755399441055744.0;
    x = fmin(fmax(x, -746.0), 800.0);
    double kf = x * (64 * 1.4426950408889634);
    kf += kShift;
    const int k = (int)__double_as_longlong(kf);
    const double kd = kf - kShift;
    double r = fma(kd, -6.93147180369123816490e-01 / 64, x);
    r = fma(kd, -1.90821492927058770002e-10 / 64, r);
    constexpr double a2 = kLn2 / 128 * (kLn2 / 128);          // r^6 ~ 3/2 a2 r^4 - 9/16 a2^2 r^2 on |r| <= sqrt(a2)
    double p = r * (1.0 / 120.0);
    p += 1.0 / 24.0 + 1.5 * a2 / 720.0;
    p = fma_k(p, r, 1.0 / 6.0);
    p = fma_k(p, r, 0.5 - 0.5625 * a2 * a2 / 720.0);
    p = fma(p, r, 1.0);
    const double t = tab.v[k & 63];
    return ldexp(fma(t, fma(p, r, (double)tab.rest[k & 63]), t), k >> 6);
}
// exp(x) for the shift eta (q - p), which is tiny for all but the heaviest tokens: a polynomial up to 2^-6,
// economised in the same way (x^7/5040 would leave 5e-17).  Which form a lane takes depends on its x alone, so the result
// does not depend on its wave.
__device__ __forceinline__ double exp_shift(double x, const Exp2& tab)
{
    constexpr double a2 = 0.015625 * 0.015625;                // x^7 ~ 7/4 a2 x^5 - 7/8 a2^2 x^3 on |x| <= sqrt(a2)
    double p = x * (1.0 / 720.0);
    p += 1.0 / 120.0 + 1.75 * a2 / 5040.0;
    p = fma_k(p, x, 1.0 / 24.0);
    p = fma_k(p, x, 1.0 / 6.0 - 0.875 * a2 * a2 / 5040.0);
    p = fma(p, x, 0.5);
    p = fma(p, x, 1.0);
    p = fma(p, x, 1.0);
    const bool large = !(fabs(x) <= 0.015625);
    if (__any(large)) {
        const double full = exp_tab(x, tab);
        p = large ? full : p;
    }
    return p;
}

}  // namespace
