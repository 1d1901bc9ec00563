// Device building blocks of the fused RD3Q41 update: node decoding and the
// periodic two-sublattice pull map (Sec. IV), moments (Sec. II), the exact
// entropic equilibrium through the closed-form shell partition function
// (Sec. V), and the storage encodings.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cmath>
#include <cstring>

#include "lattice.hpp"

namespace lbm {

// ---------------------------------------------------------------------------
// Division by a run-time invariant divisor: n / d = (umulhi(n, m) + n) >> l
// with l = ceil(log2 d) and m = floor(2^32 (2^l - d) / d) + 1, exact for all
// 32-bit n (Granlund and Montgomery, "Division by invariant integers using
// multiplication", 1994).
// ---------------------------------------------------------------------------
struct FastDiv {
    uint32_t d, m, l;
};

inline FastDiv make_fastdiv(uint32_t d)
{
    uint32_t l = 0;
    while ((uint64_t(1) << l) < d) ++l;
    uint64_t m = ((uint64_t(1) << 32) * ((uint64_t(1) << l) - d)) / d + 1;
    return FastDiv{d, uint32_t(m), l};
}

__host__ __device__ inline uint32_t umulhi32(uint32_t a, uint32_t b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __umulhi(a, b);
#else
    return uint32_t((uint64_t(a) * b) >> 32);
#endif
}

__host__ __device__ inline uint32_t fdiv(uint32_t n, const FastDiv& f)
{
    uint32_t t = umulhi32(n, f.m);
    return uint32_t((uint64_t(t) + n) >> f.l);
}

// ---------------------------------------------------------------------------
// Box geometry and the pull map.
// ---------------------------------------------------------------------------
struct Geom {
    uint32_t nx, ny, nz;
    uint32_t nxy;    // nx*ny
    uint32_t plane;  // nx*ny*nz, nodes of one sublattice
    uint32_t N;      // 2*plane
    uint32_t qs;     // elements from one q-block of the box to the next (>= N)
    FastDiv dx, dy, dz;
};

inline Geom make_geom(uint32_t nx, uint32_t ny, uint32_t nz)
{
    Geom g;
    g.nx = nx; g.ny = ny; g.nz = nz;
    g.nxy = nx * ny;
    g.plane = nx * ny * nz;
    g.N = 2 * g.plane;
    g.qs = g.N;
    g.dx = make_fastdiv(nx);
    g.dy = make_fastdiv(ny);
    g.dz = make_fastdiv(nz);
    return g;
}

struct Coord {
    uint32_t x, y, z, s;
};

__device__ inline Coord decode(uint32_t n, const Geom& g)
{
    Coord c;
    uint32_t r = fdiv(n, g.dx);
    c.x = n - r * g.nx;
    uint32_t r2 = fdiv(r, g.dy);
    c.y = r - r2 * g.ny;
    c.s = fdiv(r2, g.dz);
    c.z = r2 - c.s * g.nz;
    return c;
}

// Wrapped neighbour offsets of one node, scaled by `unit` (1 for node ids,
// sizeof(element) for byte offsets into a q-block). For an integer move by d
// in [-2, 2] along an axis the source coordinate is (x - d) mod n, held in
// o[2 - d]; i.e. o[k] = ((x + k - 2) mod n) * stride. The half moves sigma/2
// (sigma = +-1) connect the sublattices: a node at x + s/2 receives from the
// other sublattice at x + s - (1 + sigma)/2, held in h[0] for sigma = +1 and
// h[1] for sigma = -1.
struct Nbr {
    uint32_t xo[5], yo[5], zo[5];
    uint32_t xh[2], yh[2], zh[2];
    uint32_t so, sh;  // own and opposite sublattice offsets
};

// Each neighbour follows from the one before it by an add and a select (the
// wrap as a compare of offsets): one half-rate multiply per axis instead of
// five. Not for the wall kernels (MULS), where the chain of selects costs more
// than the multiplies: BF16 with walls 256^3 1134 -> 1122 us per step with
// them, 128^3 143.1 -> 140.6; FP32, FP64 and FP16 the same within 1%.
template <bool MULS = false>
__device__ inline void axis_wrap(uint32_t x, uint32_t n, uint32_t stride, uint32_t s, uint32_t o[5], uint32_t h[2])
{
    if constexpr (MULS) {
        const uint32_t m1 = x == 0 ? n - 1 : x - 1, m2 = m1 == 0 ? n - 1 : m1 - 1;
        const uint32_t p1 = x + 1 == n ? 0 : x + 1, p2 = p1 + 1 == n ? 0 : p1 + 1;
        o[0] = m2 * stride;
        o[1] = m1 * stride;
        o[2] = x * stride;
        o[3] = p1 * stride;
        o[4] = p2 * stride;
    } else {
        const uint32_t top = (n - 1) * stride;
        o[2] = x * stride;
        o[1] = o[2] == 0 ? top : o[2] - stride;
        o[0] = o[1] == 0 ? top : o[1] - stride;
        o[3] = o[2] == top ? 0 : o[2] + stride;
        o[4] = o[3] == top ? 0 : o[3] + stride;
    }
    h[0] = s ? o[2] : o[1];
    h[1] = s ? o[3] : o[2];
}

template <bool MULS = false>
__device__ inline void make_nbr(const Geom& g, const Coord& c, Nbr& nb, uint32_t unit = 1)
{
    axis_wrap<MULS>(c.x, g.nx, unit, c.s, nb.xo, nb.xh);
    axis_wrap<MULS>(c.y, g.ny, g.nx * unit, c.s, nb.yo, nb.yh);
    axis_wrap<MULS>(c.z, g.nz, g.nxy * unit, c.s, nb.zo, nb.zh);
    nb.so = c.s ? g.plane * unit : 0;
    nb.sh = c.s ? 0 : g.plane * unit;
}

// Offset (in the unit of make_nbr) of the node that population q is pulled
// from (Sec. IV: streaming along the links of the bcc lattice, periodic).
template <int q>
__device__ inline uint32_t pull_src(const Nbr& nb)
{
    constexpr HalfVel v = VEL[q];
    if constexpr (v.shell == 5) {
        return nb.sh + nb.zh[v.z > 0 ? 0 : 1] + nb.yh[v.y > 0 ? 0 : 1] + nb.xh[v.x > 0 ? 0 : 1];
    } else {
        return nb.so + nb.zo[2 - v.z / 2] + nb.yo[2 - v.y / 2] + nb.xo[2 - v.x / 2];
    }
}

// pull_src split into the part that does not depend on x (sublattice, y
// and z moves; the same for every node of an x-row) and the move along x:
// the node at x pulls population q from x + pull_dx<q>(s) (periodic) of the
// row at offset pull_row<q>.
template <int q>
__device__ inline uint32_t pull_row(const Nbr& nb)
{
    constexpr HalfVel v = VEL[q];
    if constexpr (v.shell == 5) return nb.sh + nb.zh[v.z > 0 ? 0 : 1] + nb.yh[v.y > 0 ? 0 : 1];
    else return nb.so + nb.zo[2 - v.z / 2] + nb.yo[2 - v.y / 2];
}
template <int q>
__device__ inline int pull_dx(uint32_t s)
{
    constexpr HalfVel v = VEL[q];
    if constexpr (v.shell == 5) return v.x > 0 ? (s ? 0 : -1) : (s ? 1 : 0);
    else return -(v.x / 2);
}

// ---------------------------------------------------------------------------
// Arithmetic helpers per compute type.
// ---------------------------------------------------------------------------
// The equilibrium and collision code below is __host__ __device__ so that
// the library can run the very same arithmetic on the host for testing;
// only these two helpers differ (hardware exp/reciprocal on the device).
template <typename R> __host__ __device__ inline R d_exp(R x);
template <> __host__ __device__ inline float d_exp<float>(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __expf(x);
#else
    return std::exp(x);
#endif
}
template <> __host__ __device__ inline double d_exp<double>(double x) { return exp(x); }

template <typename R> __host__ __device__ inline R d_rcp(R x);
template <> __host__ __device__ inline float d_rcp<float>(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rcpf(x);
#else
    return 1.0f / x;
#endif
}
template <> __host__ __device__ inline double d_rcp<double>(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    // the hardware's estimate and two Newton steps: within one rounding of
    // 1/x in the normal range, in 5 instructions instead of the 11 of an
    // IEEE division (which also scales for the range's ends)
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
#else
    return 1.0 / x;
#endif
}

// 1/x and a/x of the equilibrium solve, rounded as the IEEE operations round
// where x and the result are normal numbers (an estimate, Newton steps, and for
// the quotient its remainder added back), in half their instructions: FP32
// starts from the hardware's 1 ulp, FP64 from d_rcp. Against the compiler's
// division on gfx950, no difference in: the reciprocals of every FP32 mantissa
// at seven exponents (that of all ones, which Newton steps from an estimate off
// by one ulp would misround, comes out right with the hardware's); 2^29 random
// FP32 quotients and all 2^23 numerators over 0.99999994; 2^27 random FP64
// reciprocals and quotients. At 0 and infinity the result is NaN where division
// gives infinity and 0; a node that gets there is flagged either way.
template <typename R> __host__ __device__ inline R d_inv(R x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    R r = d_rcp<R>(x);
    if constexpr (sizeof(R) == 4) {
        r = fma(fma(-x, r, R(1)), r, r);
        r = fma(fma(-x, r, R(1)), r, r);
    }
    return r;
#else
    return R(1) / x;
#endif
}
template <typename R> __host__ __device__ inline R d_div(R a, R x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const R r = d_inv<R>(x), q = a * r;
    return fma(fma(-x, q, a), r, q);
#else
    return a / x;
#endif
}

// ---------------------------------------------------------------------------
// Exact entropic equilibrium (Sec. V), in deviation form.
//
// With f_eq,i = rho w_i e^{b.c_i - g c_i^2} / Z(b, g) and
// Z = sum_i w_i e^{b.c_i - g c_i^2} (the paper's beta = -b, gamma = g,
// alpha = ln Z), mass holds by construction and momentum and energy require
//     d lnZ / d b = u,   -d lnZ / d g = u^2 + 3 theta.
// Z sums in closed form over the six shells (cosh/sinh of b_a/2, b_a, 2 b_a
// and powers of t = e^{-g/4}). Newton minimises the convex function
// lnZ - b.u + g (u^2 + 3 theta), whose Hessian is the 4x4 covariance of
// (c, -c^2) under the equilibrium. Start: the continuous Maxwellian,
// b = u/theta, g = 1/(2 theta) - 1/(2 theta0).
//
// Everything that decides conservation is carried as a deviation from the
// reference state w_i rho_ref (whose multipliers are zero): e^{b.c - g c^2}
// - 1 is formed from sinh and cosh - 1 of the multipliers and expm1 of the
// temperature multiplier, never as a difference of two numbers near one.
// The normalisation enters as kappa with rho/Z = rho_ref (1 + kappa), so a
// collision conserves mass, momentum and energy to the rounding of small
// quantities, whatever the rounding of the weights themselves.
// ---------------------------------------------------------------------------
template <typename R>
struct Mult {
    R b[3];
    R g;
};

// One Horner step x p + c with a literal c. Written out in FP32: left to
// itself the compiler moves most of the constants into registers first (36
// more instructions in the step kernel).
#if defined(__HIP_DEVICE_COMPILE__)
template <uint32_t C>
__device__ inline float horner_bits(float x, float p)
{
    float r;
    asm("v_fmaak_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(p), "n"(C));
    return r;
}
#define LBM_HORNER(x, p, c) horner_bits<__builtin_bit_cast(uint32_t, float(c))>(x, p)
#else
#define LBM_HORNER(x, p, c) fmaf(x, p, float(c))
#endif

// sinh(x) and cosh(x) - 1, accurate for small |x| (Taylor series to the
// precision of R for |x| <= 1, exponentials beyond).
template <typename R>
__host__ __device__ inline void hyp(R x, R& sh, R& chm)
{
    const R x2 = x * x;
    if constexpr (sizeof(R) == 4) {
        R ps = LBM_HORNER(x2, R(1.0 / 39916800), 1.0 / 362880);   // 1/11!, 1/9!
        R pc = LBM_HORNER(x2, R(1.0 / 479001600), 1.0 / 3628800);  // 1/12!, 1/10!
        ps = LBM_HORNER(x2, ps, 1.0 / 5040);
        pc = LBM_HORNER(x2, pc, 1.0 / 40320);
        ps = LBM_HORNER(x2, ps, 1.0 / 120);
        pc = LBM_HORNER(x2, pc, 1.0 / 720);
        ps = LBM_HORNER(x2, ps, 1.0 / 6);
        pc = LBM_HORNER(x2, pc, 1.0 / 24);
        sh = x * fma(x2, ps, R(1));
        chm = x2 * fma(x2, pc, R(0.5));
    } else {
        R ps = R(1.0 / 121645100408832000.0);  // 1/19!
        R pc = R(1.0 / 2432902008176640000.0); // 1/20!
        ps = R(1.0 / 355687428096000.0) + x2 * ps;      // 1/17!
        pc = R(1.0 / 6402373705728000.0) + x2 * pc;     // 1/18!
        ps = R(1.0 / 1307674368000.0) + x2 * ps;        // 1/15!
        pc = R(1.0 / 20922789888000.0) + x2 * pc;       // 1/16!
        ps = R(1.0 / 6227020800.0) + x2 * ps;           // 1/13!
        pc = R(1.0 / 87178291200.0) + x2 * pc;          // 1/14!
        ps = R(1.0 / 39916800.0) + x2 * ps;             // 1/11!
        pc = R(1.0 / 479001600.0) + x2 * pc;            // 1/12!
        ps = R(1.0 / 362880.0) + x2 * ps;               // 1/9!
        pc = R(1.0 / 3628800.0) + x2 * pc;              // 1/10!
        ps = R(1.0 / 5040.0) + x2 * ps;                 // 1/7!
        pc = R(1.0 / 40320.0) + x2 * pc;                // 1/8!
        ps = R(1.0 / 120.0) + x2 * ps;                  // 1/5!
        pc = R(1.0 / 720.0) + x2 * pc;                  // 1/6!
        ps = R(1.0 / 6.0) + x2 * ps;                    // 1/3!
        pc = R(1.0 / 24.0) + x2 * pc;                   // 1/4!
        sh = x * (R(1) + x2 * ps);
        chm = x2 * (R(0.5) + x2 * pc);
    }
    if (__builtin_expect(x2 > R(1), 0)) {
        const R ep = d_exp<R>(x), em = d_exp<R>(-x);
        sh = R(0.5) * (ep - em);
        chm = R(0.5) * (ep + em) - R(1);
    }
}

// e^y - 1, accurate for small |y| (series for |y| <= 1/2, exponential beyond).
template <typename R>
__host__ __device__ inline R expm1_dev(R y)
{
    R p;
    if constexpr (sizeof(R) == 4) {
        p = R(1.0 / 362880);
        p = R(1.0 / 40320) + y * p;
        p = R(1.0 / 5040) + y * p;
        p = R(1.0 / 720) + y * p;
        p = R(1.0 / 120) + y * p;
        p = R(1.0 / 24) + y * p;
        p = R(1.0 / 6) + y * p;
        p = R(0.5) + y * p;
    } else {
        p = R(1.0 / 6402373705728000.0);  // 1/18!
        const double inv_fact[] = {1.0 / 355687428096000.0, 1.0 / 20922789888000.0, 1.0 / 1307674368000.0,
                                   1.0 / 87178291200.0, 1.0 / 6227020800.0, 1.0 / 479001600.0, 1.0 / 39916800.0,
                                   1.0 / 3628800.0, 1.0 / 362880.0, 1.0 / 40320.0, 1.0 / 5040.0, 1.0 / 720.0,
                                   1.0 / 120.0, 1.0 / 24.0, 1.0 / 6.0, 0.5};
#pragma unroll
        for (int i = 0; i < 16; ++i) p = R(inv_fact[i]) + y * p;
    }
    R r = y + y * y * p;
    if (__builtin_expect(y * y > R(0.25), 0)) r = d_exp<R>(y) - R(1);
    return r;
}

// (1 + a)(1 + b) - 1
template <typename R>
__host__ __device__ inline R dmul(R a, R b)
{
    return fma(a, b, a + b);
}

// Shell structure of the Gibbs factors at multipliers (b, g).
template <typename R>
struct Shells {
    // per axis: sinh and cosh-1 of b/2, b and 2b
    R sh[3], chm[3], s1[3], c1m[3], s2[3], c2m[3];
    // t^k - 1 for t = e^{-g/4}, the shell exponents k = 4|c|^2: 3, 4, 8, 12, 16
    R tau[6];  // indexed by shell (tau[0] = 0 for the rest velocity)
    R zdev[6]; // shell contributions to Z - sum_i w_i
    R zeta;    // Z - sum_i w_i
    R Z;
};

// |c|^2 of each shell as stored with R: 0, 1, 4, 2, 3, 3/4.
template <typename R>
__host__ __device__ inline void shells_at(const Mult<R>& m, Shells<R>& S)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        hyp<R>(R(0.5) * m.b[a], S.sh[a], S.chm[a]);
        S.s1[a] = R(2) * S.sh[a] * (R(1) + S.chm[a]);  // sinh b
        S.c1m[a] = R(2) * S.sh[a] * S.sh[a];           // cosh b - 1
        S.s2[a] = R(2) * S.s1[a] * (R(1) + S.c1m[a]);  // sinh 2b
        S.c2m[a] = R(2) * S.s1[a] * S.s1[a];           // cosh 2b - 1
    }
    const R t1 = expm1_dev<R>(R(-0.25) * m.g);
    const R t2 = dmul(t1, t1), t3 = dmul(t2, t1), t4 = dmul(t2, t2), t8 = dmul(t4, t4), t12 = dmul(t8, t4),
            t16 = dmul(t8, t8);
    S.tau[0] = R(0);
    S.tau[1] = t4;
    S.tau[2] = t16;
    S.tau[3] = t8;
    S.tau[4] = t12;
    S.tau[5] = t3;
    // shell sums of the axis factors, as deviations from their value at b = 0
    const R sc1 = S.c1m[0] + S.c1m[1] + S.c1m[2];                         // sum (cosh b - 1)
    const R sc2 = S.c2m[0] + S.c2m[1] + S.c2m[2];                         // sum (cosh 2b - 1)
    const R pxy = dmul(S.c1m[0], S.c1m[1]), pxz = dmul(S.c1m[0], S.c1m[2]), pyz = dmul(S.c1m[1], S.c1m[2]);
    const R p3 = dmul(pxy, S.c1m[2]);                                     // prod cosh b - 1
    const R h3 = dmul(dmul(S.chm[0], S.chm[1]), S.chm[2]);                // prod cosh b/2 - 1
    S.zdev[0] = R(0);
    S.zdev[1] = R(2 * W_SC1) * (R(3) * t4 + (R(1) + t4) * sc1);
    S.zdev[2] = R(2 * W_SC2) * (R(3) * t16 + (R(1) + t16) * sc2);
    S.zdev[3] = R(4 * W_FCC) * (R(3) * t8 + (R(1) + t8) * (pxy + pxz + pyz));
    S.zdev[4] = R(8 * W_BCC) * dmul(t12, p3);
    S.zdev[5] = R(8 * W_HALF) * dmul(t3, h3);
    S.zeta = S.zdev[1] + S.zdev[2] + S.zdev[3] + S.zdev[4] + S.zdev[5];
    S.Z = R(SUM_W) + S.zeta;
}

// Node state entering the equilibrium: deviations of the conserved sums
// from the reference state w_i rho_ref, and rho itself.
template <typename R>
struct NodeDev {
    R rho, irho;     // density and 1/rho
    R drho;          // sum_i f_i - rho_ref sum_i w_i
    R j[3];          // momentum sum_i f_i c_i
    R de2;           // sum_i f_i c_i^2 - rho_ref sum_i w_i c_i^2
    R rho_ref;
};

// kappa with rho/Z = rho_ref (1 + kappa)
template <typename R>
__host__ __device__ inline R kappa_of(const NodeDev<R>& st, const Shells<R>& S)
{
    return d_div<R>(st.drho - st.rho_ref * S.zeta, st.rho_ref * S.Z);
}

// One Newton step on the multipliers. ENERGY: the five constraints of the
// energy-conserving equilibrium (unknowns b and g); otherwise mass and
// momentum only (the isothermal equilibrium: unknowns b, g stays 0).
// Returns the squared length of the step.
template <typename R, bool ENERGY = true>
__host__ __device__ inline R newton_step(Mult<R>& m, const NodeDev<R>& st)
{
    Shells<R> S;
    shells_at<R>(m, S);
    const R T1 = R(W_SC1) * (R(1) + S.tau[1]), T2 = R(W_SC2) * (R(1) + S.tau[2]),
            T3 = R(W_FCC) * (R(1) + S.tau[3]), T4 = R(W_BCC) * (R(1) + S.tau[4]),
            T5 = R(W_HALF) * (R(1) + S.tau[5]);
    R C1[3], Ch[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        C1[a] = R(1) + S.c1m[a];
        Ch[a] = R(1) + S.chm[a];
    }
    const R Z = S.Z, iz = d_inv<R>(Z);
    // <c^2> Z = sum_s |c_s|^2 (shell part of Z); its deviation is eta2
    const R eta2 = S.zdev[1] + R(4) * S.zdev[2] + R(2) * S.zdev[3] + R(3) * S.zdev[4] + R(0.75) * S.zdev[5];
    const R N2 = R(SUM_WC2) + eta2;
    // Z-weighted moments for the Hessian
    const R sc1 = R(2) * T1 * (C1[0] + C1[1] + C1[2]);
    const R sc2 = R(2) * T2 * (R(3) + S.c2m[0] + S.c2m[1] + S.c2m[2]);
    const R fcc = R(4) * T3 * (C1[0] * C1[1] + C1[0] * C1[2] + C1[1] * C1[2]);
    const R bcc = R(8) * T4 * (C1[0] * C1[1] * C1[2]);
    const R hlf = R(8) * T5 * (Ch[0] * Ch[1] * Ch[2]);
    const R N4 = sc1 + R(16) * sc2 + R(4) * fcc + R(9) * bcc + R(0.5625) * hlf;
    R M[3], XX[3], XC[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int b = (a + 1) % 3, c = (a + 2) % 3;
        const R s1 = R(2) * T1 * S.s1[a];
        const R s2 = R(4) * T2 * S.s2[a];
        const R f = R(4) * T3 * S.s1[a] * (C1[b] + C1[c]);
        const R bb = R(8) * T4 * S.s1[a] * C1[b] * C1[c];
        const R hh = R(4) * T5 * S.sh[a] * Ch[b] * Ch[c];
        M[a] = s1 + s2 + f + bb + hh;                                   // Z <c_a>
        XC[a] = s1 + R(4) * s2 + R(2) * f + R(3) * bb + R(0.75) * hh;   // Z <c_a c^2>
        XX[a] = R(2) * T1 * C1[a] + R(8) * T2 * (R(1) + S.c2m[a]) + R(4) * T3 * C1[a] * (C1[b] + C1[c]) + bcc +
                R(0.25) * hlf;                                          // Z <c_a^2>
    }
    const R XYxy = R(4) * T3 * S.s1[0] * S.s1[1] + R(8) * T4 * S.s1[0] * S.s1[1] * C1[2] +
                   R(2) * T5 * S.sh[0] * S.sh[1] * Ch[2];
    const R XYxz = R(4) * T3 * S.s1[0] * S.s1[2] + R(8) * T4 * S.s1[0] * S.s1[2] * C1[1] +
                   R(2) * T5 * S.sh[0] * S.sh[2] * Ch[1];
    const R XYyz = R(4) * T3 * S.s1[1] * S.s1[2] + R(8) * T4 * S.s1[1] * S.s1[2] * C1[0] +
                   R(2) * T5 * S.sh[1] * S.sh[2] * Ch[0];

    // gradient of lnZ - b.u + g (u^2 + 3 theta), formed from deviations:
    //   rho (<c> - u)             = rho_ref (1 + kappa) Z<c> - j
    //   rho (u^2 + 3 theta - <c^2>) = de2 - rho_ref (eta2 + kappa (sum w c^2 + eta2))
    const R kap = kappa_of<R>(st, S);
    const R r0 = (st.rho_ref * (R(1) + kap) * M[0] - st.j[0]) * st.irho;
    const R r1 = (st.rho_ref * (R(1) + kap) * M[1] - st.j[1]) * st.irho;
    const R r2 = (st.rho_ref * (R(1) + kap) * M[2] - st.j[2]) * st.irho;
    if constexpr (!ENERGY) {
        // 3x3 covariance of c under the equilibrium, LDL^T solve
        const R mu0 = M[0] * iz, mu1 = M[1] * iz, mu2 = M[2] * iz;
        const R H00 = XX[0] * iz - mu0 * mu0, H11 = XX[1] * iz - mu1 * mu1, H22 = XX[2] * iz - mu2 * mu2;
        const R H10 = XYxy * iz - mu1 * mu0, H20 = XYxz * iz - mu2 * mu0, H21 = XYyz * iz - mu2 * mu1;
        const R iD0 = d_rcp<R>(H00);
        const R l10 = H10 * iD0, l20 = H20 * iD0;
        const R D1 = H11 - l10 * H10, iD1 = d_rcp<R>(D1);
        const R l21 = (H21 - l20 * H10) * iD1;
        const R D2 = H22 - l20 * H20 - l21 * l21 * D1, iD2 = d_rcp<R>(D2);
        const R y0 = r0, y1 = r1 - l10 * y0, y2 = r2 - l20 * y0 - l21 * y1;
        const R x2 = y2 * iD2;
        const R x1 = y1 * iD1 - l21 * x2;
        const R x0 = y0 * iD0 - l10 * x1 - l20 * x2;
        m.b[0] -= x0;
        m.b[1] -= x1;
        m.b[2] -= x2;
        return x0 * x0 + x1 * x1 + x2 * x2;
    }
    const R r3 = (st.de2 - st.rho_ref * (eta2 + kap * N2)) * st.irho;

    const R mu0 = M[0] * iz, mu1 = M[1] * iz, mu2 = M[2] * iz, m2 = N2 * iz;
    const R H00 = XX[0] * iz - mu0 * mu0, H11 = XX[1] * iz - mu1 * mu1, H22 = XX[2] * iz - mu2 * mu2;
    const R H10 = XYxy * iz - mu1 * mu0, H20 = XYxz * iz - mu2 * mu0, H21 = XYyz * iz - mu2 * mu1;
    const R H30 = m2 * mu0 - XC[0] * iz, H31 = m2 * mu1 - XC[1] * iz, H32 = m2 * mu2 - XC[2] * iz;
    const R H33 = N4 * iz - m2 * m2;

    // LDL^T factorisation and solve of H d = r
    const R D0 = H00, iD0 = d_rcp<R>(D0);
    const R l10 = H10 * iD0, l20 = H20 * iD0, l30 = H30 * iD0;
    const R D1 = H11 - l10 * H10, iD1 = d_rcp<R>(D1);
    const R l21 = (H21 - l20 * H10) * iD1, l31 = (H31 - l30 * H10) * iD1;
    const R D2 = H22 - l20 * H20 - l21 * l21 * D1, iD2 = d_rcp<R>(D2);
    const R l32 = (H32 - l30 * H20 - l31 * l21 * D1) * iD2;
    const R D3 = H33 - l30 * H30 - l31 * l31 * D1 - l32 * l32 * D2, iD3 = d_rcp<R>(D3);
    const R y0 = r0, y1 = r1 - l10 * y0, y2 = r2 - l20 * y0 - l21 * y1, y3 = r3 - l30 * y0 - l31 * y1 - l32 * y2;
    const R x3 = y3 * iD3;
    const R x2 = y2 * iD2 - l32 * x3;
    const R x1 = y1 * iD1 - l21 * x2 - l31 * x3;
    const R x0 = y0 * iD0 - l10 * x1 - l20 * x2 - l30 * x3;
    m.b[0] -= x0;
    m.b[1] -= x1;
    m.b[2] -= x2;
    m.g -= x3;
    return x0 * x0 + x1 * x1 + x2 * x2 + x3 * x3;
}

// ---------------------------------------------------------------------------
// Series equilibrium E1 (Sec. V): f_eq,i = w_i rho f~_i(eta) P_i(u), with
// the zero-velocity series to third order in eta = theta/theta0 - 1,
//   f~ = 1 + eta/2 (x - 3) + eta^2/8 (x^2 - 10 x + 15)
//          + eta^3/48 (x^3 - 21 x^2 + 105 x - 105),   x = c^2/theta0,
// and the cubic velocity polynomial with uc = u.c/theta,
//   P = 1 + uc + uc^2/2 + uc^3/6 - u^2/(2 theta) (1 - A1)
//       - u^2 c^2 A1/(6 theta^2) + u^2 uc A2/(6 theta) - u^2 c^2 uc A1/(6 theta^2),
//   A1 = (5/2) M2 / (1 + (5/2) M2),  A2 = 5 A1 (1 - M2) - (3 + M2' - 5 M2),
// where M2, M2' are the relative errors of the fourth moments of f~ (sums
// over the lattice). In deviation form eps_i = f~ P - 1 = dmul(T_s, Q_i),
// T_s = f~ - 1 per shell and Q_i = P_i - 1 = alpha_s + uc (1 + beta_s +
// uc (1/2 + uc/6)).
// ---------------------------------------------------------------------------
template <typename R>
struct SeriesCoef {
    R a[3];        // u / theta
    R T[6];        // f~ - 1 per shell
    R alpha[6];    // u-independent part of P - 1 per shell
    R beta1[6];    // 1 + coefficient of uc u^2 per shell
};

__host__ __device__ constexpr double series_k(int s, int order)
{
    const double x = SHELL_C2[s] / THETA0;
    return order == 1 ? 0.5 * (x - 3.0)
         : order == 2 ? (x * x - 10.0 * x + 15.0) / 8.0
                      : (x * x * x - 21.0 * x * x + 105.0 * x - 105.0) / 48.0;
}

// eta = theta/theta0 - 1 is passed in (formed from moment deviations by
// the caller, free of the cancellation of theta/theta0 - 1).
template <typename R>
__host__ __device__ inline void series_coef(R ux, R uy, R uz, R eta, SeriesCoef<R>& sc)
{
    const R theta = R(THETA0) * (R(1) + eta);
    R s4 = R(0), sxy = R(0);
#pragma unroll
    for (int s = 0; s < 6; ++s) {
        sc.T[s] = eta * (R(series_k(s, 1)) + eta * (R(series_k(s, 2)) + eta * R(series_k(s, 3))));
        s4 += R(SHELL_C4[s] / (15.0 * THETA0 * THETA0)) * sc.T[s];
        sxy += R(SHELL_CXCY[s] / (THETA0 * THETA0)) * sc.T[s];
    }
    // M2 = sum w c^4 (1 + T)/(15 theta^2) - 1 and M2' likewise, formed from
    // the reference-state values (exact lattice sums) and the deviations
    constexpr double M20 = (SHELL_C4[0] + SHELL_C4[1] + SHELL_C4[2] + SHELL_C4[3] + SHELL_C4[4] + SHELL_C4[5]) /
                           (15.0 * THETA0 * THETA0) - 1.0;
    constexpr double MXY0 = (SHELL_CXCY[0] + SHELL_CXCY[1] + SHELL_CXCY[2] + SHELL_CXCY[3] + SHELL_CXCY[4] +
                             SHELL_CXCY[5]) / (THETA0 * THETA0) - 1.0;
    const R ie2 = R(1) / ((R(1) + eta) * (R(1) + eta));
    const R de = eta * (R(2) + eta);
    const R M2 = (R(M20) + s4 - de) * ie2;
    const R M2p = (R(MXY0) + sxy - de) * ie2;
    const R A1 = R(2.5) * M2 / (R(1) + R(2.5) * M2);
    const R A2 = R(5) * A1 * (R(1) - M2) - (R(3) + M2p - R(5) * M2);
    const R ith = R(1) / theta;
    sc.a[0] = ux * ith;
    sc.a[1] = uy * ith;
    sc.a[2] = uz * ith;
    const R U = (ux * ux + uy * uy + uz * uz) * ith;  // u^2 / theta
    const R uA1 = U * A1 * ith * R(1.0 / 6.0);        // u^2 A1 / (6 theta^2)
#pragma unroll
    for (int s = 0; s < 6; ++s) {
        sc.alpha[s] = -R(0.5) * U * (R(1) - A1) - uA1 * R(SHELL_C2[s]);
        sc.beta1[s] = R(1) + U * A2 * R(1.0 / 6.0) - uA1 * R(SHELL_C2[s]);
    }
}

// eps_q = f~ P - 1 for velocity q
template <int q, typename R>
__host__ __device__ inline R series_eps(const SeriesCoef<R>& sc)
{
    constexpr HalfVel v = VEL[q];
    constexpr int s = v.shell;
    if constexpr (s == 0) {
        return dmul(sc.T[0], sc.alpha[0]);
    } else {
        R uc = R(0);
        if constexpr (v.x != 0) uc = fma(sc.a[0], R(0.5 * v.x), uc);
        if constexpr (v.y != 0) uc = fma(sc.a[1], R(0.5 * v.y), uc);
        if constexpr (v.z != 0) uc = fma(sc.a[2], R(0.5 * v.z), uc);
        R t = fma(uc, R(1.0 / 6.0), R(0.5));
        t = fma(uc, t, sc.beta1[s]);
        const R Qd = fma(uc, t, sc.alpha[s]);
        return dmul(sc.T[s], Qd);
    }
}

// e^{b.c_q - g c_q^2} - 1 for velocity q, from the shell structure.
template <int q, typename R>
__host__ __device__ inline R gibbs_dev(const Shells<R>& S)
{
    constexpr HalfVel v = VEL[q];
    auto fac = [&](int a, int h) -> R {
        switch (h) {
            case 1: return S.chm[a] + S.sh[a];
            case -1: return S.chm[a] - S.sh[a];
            case 2: return S.c1m[a] + S.s1[a];
            case -2: return S.c1m[a] - S.s1[a];
            case 4: return S.c2m[a] + S.s2[a];
            case -4: return S.c2m[a] - S.s2[a];
            default: return R(0);
        }
    };
    R e = S.tau[v.shell];
    if constexpr (v.x != 0) e = dmul(e, fac(0, v.x));
    if constexpr (v.y != 0) e = dmul(e, fac(1, v.y));
    if constexpr (v.z != 0) e = dmul(e, fac(2, v.z));
    return e;
}

// ---------------------------------------------------------------------------
// Moments of 41 values by shell: for each shell s the plain sum and the sums
// signed by the sign of c_x, c_y, c_z (the magnitude |c_a| of a shell is
// applied by the caller). The two 8-velocity shells use a butterfly.
// ---------------------------------------------------------------------------
template <typename R>
struct ShellSums {
    R s0[6], sx[6], sy[6], sz[6];
};

// v(q) gives value q; its type's + and - give an R (the values themselves, or
// 16-bit inputs converted in the same instruction).
template <int q0, typename R, class GET>
__host__ __device__ inline void cube8(const GET& v, R& s0, R& sx, R& sy, R& sz)
{
    auto x = [&](auto ic) { return v(std::integral_constant<int, q0 + decltype(ic)::value>{}); };
    using std::integral_constant;
    const auto v0 = x(integral_constant<int, 0>{});
    const auto v1 = x(integral_constant<int, 1>{});
    const auto v2 = x(integral_constant<int, 2>{});
    const auto v3 = x(integral_constant<int, 3>{});
    const auto v4 = x(integral_constant<int, 4>{});
    const auto v5 = x(integral_constant<int, 5>{});
    const auto v6 = x(integral_constant<int, 6>{});
    const auto v7 = x(integral_constant<int, 7>{});
    // order (+++), (++-), (+-+), (+--), (-++), (-+-), (--+), (---)
    const R a0 = v0 + v1, a1 = v0 - v1, a2 = v2 + v3, a3 = v2 - v3;
    const R a4 = v4 + v5, a5 = v4 - v5, a6 = v6 + v7, a7 = v6 - v7;
    const R b0 = a0 + a2, b1 = a0 - a2, b2 = a1 + a3;
    const R c0 = a4 + a6, c1 = a4 - a6, c2 = a5 + a7;
    s0 = b0 + c0;
    sx = b0 - c0;
    sy = b1 + c1;
    sz = b2 + c2;
}

// four values of one coordinate plane of the fcc shell: (+,+), (+,-), (-,+), (-,-)
template <int pp, int pm, int mp, int mm, typename R, class GET>
__host__ __device__ inline void plane4(const GET& v, R& s0, R& d1, R& d2)
{
    const auto a = v(std::integral_constant<int, pp>{});
    const auto b = v(std::integral_constant<int, pm>{});
    const auto c = v(std::integral_constant<int, mp>{});
    const auto d = v(std::integral_constant<int, mm>{});
    const R u1 = a + b, u2 = c + d, v1 = a - b, v2 = c - d;
    s0 = u1 + u2;
    d1 = u1 - u2;
    d2 = v1 + v2;
}

template <typename R, class GET>
__host__ __device__ inline void shell_sums(const GET& v, ShellSums<R>& S)
{
    S.s0[0] = R(v(std::integral_constant<int, 0>{}));
    S.sx[0] = S.sy[0] = S.sz[0] = R(0);
    // sc-1 (q 1..6) and sc-2 (q 7..12): +x, +y, +z, -z, -y, -x
    static_for<2>([&](auto kc) {
        constexpr int k = decltype(kc)::value, q = 1 + 6 * k;
        const auto xp = v(std::integral_constant<int, q>{});
        const auto yp = v(std::integral_constant<int, q + 1>{});
        const auto zp = v(std::integral_constant<int, q + 2>{});
        const auto zm = v(std::integral_constant<int, q + 3>{});
        const auto ym = v(std::integral_constant<int, q + 4>{});
        const auto xm = v(std::integral_constant<int, q + 5>{});
        S.s0[1 + k] = (xp + xm) + (yp + ym) + (zp + zm);
        S.sx[1 + k] = xp - xm;
        S.sy[1 + k] = yp - ym;
        S.sz[1 + k] = zp - zm;
    });
    // fcc-1 (q 13..24): (1,1,0) (1,0,1) (1,0,-1) (1,-1,0) (0,1,1) (0,1,-1)
    //                   (0,-1,1) (0,-1,-1) (-1,1,0) (-1,0,1) (-1,0,-1) (-1,-1,0)
    {
        R sxy, dxy_x, dxy_y, sxz, dxz_x, dxz_z, syz, dyz_y, dyz_z;
        plane4<13, 16, 21, 24>(v, sxy, dxy_x, dxy_y);
        plane4<14, 15, 22, 23>(v, sxz, dxz_x, dxz_z);
        plane4<17, 18, 19, 20>(v, syz, dyz_y, dyz_z);
        S.s0[3] = sxy + sxz + syz;
        S.sx[3] = dxy_x + dxz_x;
        S.sy[3] = dxy_y + dyz_y;
        S.sz[3] = dxz_z + dyz_z;
    }
    cube8<25>(v, S.s0[4], S.sx[4], S.sy[4], S.sz[4]);  // bcc-1
    cube8<33>(v, S.s0[5], S.sx[5], S.sy[5], S.sz[5]);  // bcc-1/2
}

// |c_a| of a nonzero component and |c|^2, per shell
constexpr double SHELL_CA[6] = {0.0, 1.0, 2.0, 1.0, 1.0, 0.5};

// ---------------------------------------------------------------------------
// Storage encodings. Every kernel works on deviations d_q = f_q - w_q rho_ref
// with rho_ref = rho0 for the shifted forms and 0 otherwise; the shifted
// forms hold h_q = d_q 2^{k_q} in 16 bits.
// ---------------------------------------------------------------------------
struct StoreF64 {
    using T = double;
    using R = double;
    static constexpr bool shifted = false;
    static constexpr bool unit_scale = true;
    static constexpr float SAT = 0.0f;  // no saturation
    __device__ static R decode(T v) { return v; }
    __device__ static T encode(R v) { return v; }
    __device__ static R load(const T* p) { return *p; }
    __device__ static void store(T* p, R v) { *p = v; }
};

struct StoreF32 {
    using T = float;
    using R = float;
    static constexpr bool shifted = false;
    static constexpr bool unit_scale = true;
    static constexpr float SAT = 0.0f;  // no saturation
    __device__ static R decode(T v) { return v; }
    __device__ static T encode(R v) { return v; }
    __device__ static R load(const T* p) { return *p; }
    __device__ static void store(T* p, R v) { *p = v; }
};

// FP32 holding the shift h = f - w rho0 (scale 1).
struct StoreF32S {
    using T = float;
    using R = float;
    static constexpr bool shifted = true;
    static constexpr bool unit_scale = true;
    static constexpr float SAT = 0.0f;  // no saturation
    __device__ static R decode(T v) { return v; }
    __device__ static T encode(R v) { return v; }
    __device__ static R load(const T* p) { return *p; }
    __device__ static void store(T* p, R v) { *p = v; }
};

// Stochastic rounding to a format with `drop` fewer mantissa bits than FP32:
// add `drop` uniformly random bits below the kept mantissa, then truncate.
// The result is representable, so the final conversion is exact, and its
// expectation equals v (away from the format's subnormal range).
__device__ inline float sr_truncate(float v, uint32_t rbits, int drop)
{
    const uint32_t mask = (1u << drop) - 1u;
    uint32_t u = __float_as_uint(v) + (rbits & mask);
    return __uint_as_float(u & ~mask);
}

struct StoreF16S {
    using T = _Float16;
    using R = float;
    static constexpr bool shifted = true;
    static constexpr bool unit_scale = false;
    __device__ static R decode(T v) { return float(v); }
    __device__ static T encode(R v) { return _Float16(v); }  // round to nearest even
    __device__ static T encode_sr(R v, uint32_t r) { return _Float16(sr_truncate(v, r, 13)); }
    // Two values with the two 16-bit halves of r: the random bits are added
    // below the kept mantissa and the pair is converted with round toward
    // zero in one instruction (the same rounding as encode_sr in the normal
    // FP16 range). Round toward zero saturates at +-65504 where rounding up
    // would leave the FP16 range; a stored magnitude of SAT is therefore
    // taken as having left the range when it is read back (the next step,
    // lbm_totals), and flagged as a non-finite result.
    __device__ static void encode_sr2(R a, R b, uint32_t r, T& oa, T& ob)
    {
        const uint32_t m = r & 0x1fff1fffu;
        const float ra = __uint_as_float(__float_as_uint(a) + (m & 0xffffu));
        const float rb = __uint_as_float(__float_as_uint(b) + (m >> 16));
        const auto h = __builtin_amdgcn_cvt_pkrtz(ra, rb);
        oa = h[0];
        ob = h[1];
    }
    static constexpr float SAT = 65504.0f;  // largest finite FP16
    __device__ static R load(const T* p) { return float(*p); }
    __device__ static void store(T* p, R v) { *p = _Float16(v); }
};

// An FP16 input of a sum, the low (HI = 0) or high half of a register, whose
// conversion to FP32 rides in the add: a + b is the mixed-precision fused
// multiply-add a 1 + b (bit for bit the sum of the converted values). Written
// out because the compiler folds a conversion only where it has one use.
template <int HI>
struct HalfIn {
    uint32_t w;
    __device__ explicit operator float() const { return float(__builtin_bit_cast(_Float16, uint16_t(w >> (16 * HI)))); }
};
template <int HA, int HB>
__device__ inline float operator+(const HalfIn<HA>& a, const HalfIn<HB>& b)
{
    float r;
    if constexpr (HA == 0 && HB == 0)
        asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a.w), "v"(b.w));
    else if constexpr (HA == 0)
        asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a.w), "v"(b.w));
    else if constexpr (HB == 0)
        asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a.w), "v"(b.w));
    else
        asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a.w), "v"(b.w));
    return r;
}
template <int HA, int HB>
__device__ inline float operator-(const HalfIn<HA>& a, const HalfIn<HB>& b)
{
    float r;
    if constexpr (HA == 0 && HB == 0)
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,0] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a.w), "v"(b.w));
    else if constexpr (HA == 0)
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a.w), "v"(b.w));
    else if constexpr (HB == 0)
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a.w), "v"(b.w));
    else
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(a.w), "v"(b.w));
    return r;
}

// bfloat16 conversions on the host: decode by a 16-bit shift, encode with
// round-to-nearest-even on the dropped 16 bits (NaN kept quiet).
inline uint16_t host_f32_to_bf16_rne(float v)
{
    uint32_t u;
    std::memcpy(&u, &v, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return uint16_t((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}
inline float host_bf16_to_f32(uint16_t b)
{
    const uint32_t u = uint32_t(b) << 16;
    float v;
    std::memcpy(&v, &u, 4);
    return v;
}

// On the device the conversion float -> __bf16 is the hardware
// round-to-nearest-even conversion of gfx950.
struct StoreBF16S {
    using T = __bf16;
    using R = float;
    static constexpr bool shifted = true;
    static constexpr bool unit_scale = false;
    __device__ static R decode(T v) { return float(v); }
    __device__ static T encode(R v) { return __bf16(v); }
    __device__ static T encode_sr(R v, uint32_t r) { return __bf16(sr_truncate(v, r, 16)); }
    // Two values with the two 16-bit halves of r: the random bits are added
    // below the kept mantissa and the upper halves are the result.
    // (BF16 keeps the FP32 exponent range: no overflow beyond FP32's own.)
    __device__ static void encode_sr2(R a, R b, uint32_t r, T& oa, T& ob)
    {
        const uint32_t ua = __float_as_uint(a) + (r & 0xffffu), ub = __float_as_uint(b) + (r >> 16);
        oa = __builtin_bit_cast(T, uint16_t(ua >> 16));
        ob = __builtin_bit_cast(T, uint16_t(ub >> 16));
    }
    static constexpr float SAT = 0.0f;  // no saturation
    __device__ static R load(const T* p) { return float(*p); }
    __device__ static void store(T* p, R v) { *p = __bf16(v); }
};

// Parameters of the step kernels (passed by value).
struct StepParams {
    Geom g;
    double omega;          // relaxation rate
    float scale[6];        // 2^{k_shell + k_amp}   (shifted storage)
    float inv_scale[6];    // 2^{-(k_shell + k_amp)}
    float omw[6];          // omega w_shell rho0 2^{k_shell + k_amp} (shifted storage)
    double rho_ref;        // rho0 (shifted) or 0: reference of the stored values
    double e2_ref;         // sum_q w_q rho_ref c_q^2 = 3 rho_ref theta0
    uint32_t* flag;        // set to 1 when a node has rho <= 0, theta <= 0 or NaN
    uint32_t xcd_map;      // tile mapping of the launch (xcd_map in step_launch.hpp)
    uint32_t tiles;        // blocks of the launch
    uint32_t step;         // step counter and seed of the stochastic rounding
    uint32_t seed;
    uint32_t node0;        // index of the box's first node in the context (random-bit stream)
    const uint32_t* step_base;  // null, or a device counter added to step (graph replays)
    uint32_t model;        // equilibrium: 0 energy conserving (E2), 1 isothermal, 2 series (E1)
    const double* wall_dev;  // kinetic walls, lower then upper: f_w,q / w_q - 1 (41) and the kind (0 diffuse, 1 specular)
};

// Counter-based random bits for stochastic rounding: one hash per node and
// step ("lowbias32", C. Wellons, hash-prospector), then successive 32-bit
// words by a Weyl sequence, word k = h + (k + 1) * 2^32/phi (mod 2^32; the
// increment is the golden-ratio constant of multiplicative hashing, Knuth,
// TAOCP vol. 3, 6.4). Each word is the uniform hash plus a constant, so
// every rounding draws uniform bits; the words of one node and step are
// shifts of each other, which leaves each rounding unbiased. One add per
// word instead of xorshift's six shifts and xors: the 16-bit kernels with
// stochastic rounding are partly arithmetic-bound, and more so at the
// clock they settle to under sustained load.
constexpr uint32_t WEYL_STEP = 0x9e3779b9u;

__host__ __device__ inline uint32_t hash32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}

__host__ __device__ constexpr uint32_t weyl_word(uint32_t h, uint32_t k) { return h + (k + 1u) * WEYL_STEP; }

// FP32 x + d rounded stochastically: s = RN(x + d) with exact residual e
// (Fast2Sum, |x| >= |d|), then RN(s + e + (r - 1/2) ulp(s)) rounds the exact
// sum up or down with probabilities given by its position between the two
// neighbouring FP32 values (x > 0).
__device__ inline float sr_add(float x, float d, uint32_t r16)
{
    const float s = x + d;
    const float e = d - (s - x);
    const float ulp = __uint_as_float(__float_as_uint(s) & 0x7f800000u) * 0x1p-23f;
    const float z = fmaf(fmaf(float(r16 & 0xffffu), 0x1p-16f, -0.5f), ulp, e);
    return s + z;
}

}  // namespace lbm
