// Device-side closures and fluxes of the DGSEM right-hand side.
//
// Physical flux: Sec. Governing Equations, Eq. adevctive_flux.
// Two-point fluxes (Sec. Methodology, Eqs. fluxdiffcons and conssymm):
//   * Ranocha's entropy-conservative, kinetic-energy-preserving flux for the
//     perfect gas (logarithmic means of rho and rho/p);
//   * the Ducros split form (perfect gas or mixture).
// Riemann flux at faces and subcell interfaces (Eqs. riemann_problem1-3,
// finitevolumeflux): local Lax-Friedrichs with the wave-speed bound
// max(|v_L.n| + c_L|n|, |v_R.n| + c_R|n|).
// Mixture closures: Appendix, Thermodynamics (RRHO energies without the
// electronic mode) and Governing Equations, Eqs. internal_energies, eos.
#pragma once

#include "dgx_internal.h"

namespace dgx {

// a + b of two rounded terms: a product among them is not contracted into the
// sum, so that the result does not depend on their order.  The two-point
// fluxes use it wherever the two states' products meet; they are then
// bitwise symmetric, and both nodes of a pair may evaluate it.
__device__ __forceinline__ double sum2(double a, double b) {
#pragma clang fp contract(off)
    return a + b;
}

template <int DIM>
__device__ __forceinline__ double dotn(const double *a, const double *b) {
    double s = a[0] * b[0];
#pragma unroll
    for (int c = 1; c < DIM; ++c) s = fma(a[c], b[c], s);
    return s;
}

// Primitive state of one node.  For the perfect gas rs[0] is the nodal
// quantity of the split form in use (pair_quantity) where there is one.
template <int DIM, bool MIX>
struct St {
    double rho, v[DIM], p, rhoE, c;
    double rs[MIX ? kNS : 1];
};

// 1/x: hardware v_rcp_f64 estimate refined by two Newton-Raphson steps
// r <- r + r (1 - x r) (each step squares the relative error).
__device__ __forceinline__ double rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// sqrt(x) for wave-speed estimates (sound speeds, face-normal lengths) of
// positive normal-range x: hardware v_rsq_f64 estimate, one coupled
// Newton-Raphson step on (sqrt x, 1/(2 sqrt x)) and a final residual
// correction, without the range scaling and special-value handling of the
// library square root.  Both sides of an interface evaluate it on identical
// inputs, so interface fluxes stay bitwise equal.
__device__ __forceinline__ double wave_sqrt(double x) {
    const double r = __builtin_amdgcn_rsq(x);
    double g = x * r;
    double h = 0.5 * r;
    const double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    const double d = fma(-g, g, x);
    return fma(d, h, g);
}

// One step a b + c of a polynomial with a constant c, and its first step
// a c1 + c0.  The constant stays in scalar registers (opaque to the compiler's
// constant handling) and enters with a negation, which only the three-address
// form of the instruction takes.  Left to itself the compiler chooses the
// two-address form, whose addend is a vector register, and writes every
// constant there first: two more vector instructions per step (2,200 of the
// 11,000 of the entropy-conservative mixture kernel).
// fma_kv keeps the constant where it is used (inside a loop it is written
// again in each turn, by the scalar unit, instead of being held in scalar
// registers that run out).
__device__ __forceinline__ double fma_k(double a, double b, double c) {
    double k = -c;
    asm("" : "+s"(k));
    return fma(a, b, -k);
}
__device__ __forceinline__ double fma_kv(double a, double b, double c) {
    double k = -c;
    asm volatile("" : "+s"(k));
    return fma(a, b, -k);
}
__device__ __forceinline__ double poly_start(double a, double c1, double c0) { return fma(a, c1, c0); }

// Logarithmic mean (y - x)/ln(y/x) and its reciprocal.  With f = (y-x)/(y+x)
// and z = f^2, ln(y/x) = 2 atanh f, so the mean is (x+y)/(2 A(z)) with
// A(z) = atanh(sqrt z)/sqrt z = sum_n z^n/(2n+1).  Three branches by z:
//   * z < 1e-4: A to four terms, and for the mean 1/A expanded,
//     1 - z/3 - 4z^2/45 - 44z^3/945 (remainder < 1e-17 relative), which
//     saves a reciprocal;
//   * z < 1/9 (ratios y/x up to 2): 1/A and 2A as polynomials of degree 10,
//     interpolated at the Chebyshev nodes of [0, 1/9] with the value at 0 held
//     exact (relative error below 3e-18 and 7e-18 with the coefficients in
//     double; the Taylor series of the same degree reaches z = 0.02);
//   * beyond: the logarithm.
__device__ __forceinline__ double inv_atanh_ratio(double z) {
    // 1/A(z), 0 <= z <= 1/9
    double r = poly_start(z, -0.013685267223330775, -0.008103049428699534);
    r = fma_kv(r, z, -0.011397025330915855);
    r = fma_kv(r, z, -0.013487086275031281);
    r = fma_kv(r, z, -0.01678833152650204);
    r = fma_kv(r, z, -0.02179678054953089);
    r = fma_kv(r, z, -0.030194003931586527);
    r = fma_kv(r, z, -0.046560846557320394);
    r = fma_kv(r, z, -0.0888888888889008);
    r = fma_kv(r, z, -1.0 / 3.0);
    return fma_kv(r, z, 1.0);
}

__device__ __forceinline__ double atanh_ratio_x2(double z) {
    // 2 A(z), 0 <= z <= 1/9
    double r = poly_start(z, 0.16164938169471338, 0.08800317650868773);
    r = fma_kv(r, z, 0.12001155182857778);
    r = fma_kv(r, z, 0.13314135550881162);
    r = fma_kv(r, z, 0.15385570592912243);
    r = fma_kv(r, z, 0.18181789417326447);
    r = fma_kv(r, z, 0.22222222717801782);
    r = fma_kv(r, z, 0.2857142856710506);
    r = fma_kv(r, z, 0.40000000000014596);
    r = fma_kv(r, z, 2.0 / 3.0);
    return fma_kv(r, z, 2.0);
}

__device__ __forceinline__ double ln_mean(double x, double y) {
    const double s = x + y;
    const double d = y - x;
    const double d2 = d * d, s2 = s * s;
    if (d2 < 1e-4 * s2) {
        const double q = d * rcp(s);
        const double z = q * q;
        const double h = 0.5 * s;
        return fma(-h * z, fma_kv(z, poly_start(z, 44.0 / 945.0, 4.0 / 45.0), 1.0 / 3.0), h);
    }
    if (d2 < (1.0 / 9.0) * s2) {
        const double q = d * rcp(s);
        return 0.5 * s * inv_atanh_ratio(q * q);
    }
    // (the larger over the smaller, for symmetry)
    return fabs(d) * rcp(log(fmax(x, y) * rcp(fmin(x, y))));
}

__device__ __forceinline__ double inv_ln_mean(double x, double y) {
    const double s = x + y;
    const double d = y - x;
    const double d2 = d * d, s2 = s * s;
    if (d2 < 1e-4 * s2) {
        const double rs = rcp(s);
        const double q = d * rs;
        const double z = q * q;
        return fma_kv(z, fma_kv(z, poly_start(z, 2.0 / 7.0, 2.0 / 5.0), 2.0 / 3.0), 2.0) * rs;
    }
    if (d2 < (1.0 / 9.0) * s2) {
        const double rs = rcp(s);
        const double q = d * rs;
        return atanh_ratio_x2(q * q) * rs;
    }
    return log(fmax(x, y) * rcp(fmin(x, y))) * rcp(fabs(d));
}

// The same where nine of them meet in one flux (the mixture's entropy-
// conservative one): a single polynomial range, so that the usual pair takes
// no branch, and for ratios above 2 the logarithm from the quotient of the
// mantissas, ln(y/x) = k ln 2 + 2 f A(f^2) with f = (my - mx)/(my + mx),
// |f| <= 1/3: the same polynomial, without a library logarithm.  Both of them
// may be negative (the ratio counts); of opposite sign, where |f| > 1, there is
// no logarithm and the result is no number.
__device__ __forceinline__ double ln_ratio_far(double x, double y) {
    const double mx = __builtin_amdgcn_frexp_mant(x), my = __builtin_amdgcn_frexp_mant(y);
    const int k = __builtin_amdgcn_frexp_exp(y) - __builtin_amdgcn_frexp_exp(x);
    const double q = (my - mx) * rcp(my + mx);
    const double l = fma((double)k, 0.69314718055994529, q * atanh_ratio_x2(q * q));
    return fabs(q) < 1.0 ? l : (double)NAN;
}

// ln mean of densities (0 where one of them is 0, the limit)
__device__ __forceinline__ double ln_mean_wide(double x, double y) {
    const double s = x + y, d = y - x;
    const double q = d * rcp(fmax(fabs(s), 1e-300));  // up to its sign
    double m = 0.5 * s * inv_atanh_ratio(q * q);
    if (3.0 * fabs(d) > fabs(s)) m = (x == 0.0 || y == 0.0) ? 0.0 : d * rcp(ln_ratio_far(x, y));
    return m;
}

// reciprocal of the ln mean of numbers other than 0
__device__ __forceinline__ double inv_ln_mean_wide(double x, double y) {
    const double s = x + y, d = y - x, rs = rcp(s);
    const double q = d * rs;
    double m = atanh_ratio_x2(q * q) * rs;
    if (3.0 * fabs(d) > fabs(s)) m = ln_ratio_far(x, y) * rcp(d);
    return m;
}

// ---------------------------------------------------------------- mixture
// Argument reduction of the exponential: y = n ln 2 + r with |r| <= ln(2)/2;
// returns e^r - 1 to its last digits (Taylor to r^13: remainder below 4e-18
// on this range), so that e^y = 2^n (1 + p).  y is cut at +-7e8, where n still
// fits an int (so do sums of two such n) and 2^n has long under- or
// overflowed (a NaN is cut too: callers use T beside it, which carries it on).
__device__ __forceinline__ double expm1_reduced(double y, int &n) {
    y = fmin(fmax(y, -7e8), 7e8);
    // round y / ln 2 to an integer in the low bits of t
    const double t = fma(y, 1.4426950408889634, 6755399441055744.0);
    const double k = t - 6755399441055744.0;
    n = (int)(unsigned)__double_as_longlong(t);
    // ln 2 as its double and the remainder
    const double r = fma(-k, 2.3190468138462996e-17, fma(-k, 0.69314718055994529, y));
    double q = poly_start(r, 1.0 / 6227020800.0, 1.0 / 479001600.0);
    q = fma_k(q, r, 1.0 / 39916800.0);
    q = fma_k(q, r, 1.0 / 3628800.0);
    q = fma_k(q, r, 1.0 / 362880.0);
    q = fma_k(q, r, 1.0 / 40320.0);
    q = fma_k(q, r, 1.0 / 5040.0);
    q = fma_k(q, r, 1.0 / 720.0);
    q = fma_k(q, r, 1.0 / 120.0);
    q = fma_k(q, r, 1.0 / 24.0);
    q = fma_k(q, r, 1.0 / 6.0);
    q = fma_k(q, r, 0.5);
    return fma(r * r, q, r);
}

// e^-x and 1 - e^-x from one reduction, without a branch: with e^-x =
// 2^n (1 + p), 1 - e^-x = (1 - 2^n) - 2^n p, which is -p itself for small x
// (n = 0, no cancellation) and is at least 0.29 otherwise.
__device__ __forceinline__ void exp_pair(double x, double &em, double &om) {
    int n;
    const double p = expm1_reduced(-x, n);
    const double s = ldexp(1.0, n);
    em = fma(s, p, s);
    om = fma(-s, p, 1.0 - s);
}

// Which species are molecules: with STD the documented order (N2, O2, NO, N,
// O), known at compile time, so that the three vibrational terms are
// evaluated side by side; else the flags of the species table, tested one
// species after another.  MixC::std_mol says which of the two holds.
template <bool STD>
__device__ __forceinline__ bool mix_is_mol(const MixC &M, int s) {
    return STD ? s < 3 : M.mol[s] != 0;
}

// Vibrational energy sum_s rho_s R_s theta_s/(e^x - 1) and its T-derivative,
// x = theta_s/T.
template <bool STD>
__device__ __forceinline__ void mix_vib(const MixC &M, const double *rs, double T, double &ev, double &cv) {
    const double iT = rcp(T);
    ev = 0.0;
    cv = 0.0;
#pragma unroll
    for (int s = 0; s < kNS; ++s) {
        if (mix_is_mol<STD>(M, s)) {
            const double x = M.thv[s] * iT;
            double em, om;  // e^-x, 1 - e^-x
            exp_pair(x, em, om);
            // R theta/(e^x - 1) = R theta e^-x / (1 - e^-x); its T-derivative R x^2 e^-x / (1 - e^-x)^2
            const double io = rcp(om);
            const double q = em * io;
            const double c = rs[s] * M.Rs[s];
            ev = fma(c * M.thv[s], q, ev);
            cv = fma(c * x * x, q * io, cv);
        }
    }
}

// Heat capacity density without vibration: 3/2 R_s per atom, 5/2 R_s per
// linear molecule.
template <bool STD>
__device__ __forceinline__ double mix_cv_rigid(const MixC &M, const double *rs) {
    double a = 0.0;
#pragma unroll
    for (int s = 0; s < kNS; ++s) a = fma(rs[s], mix_is_mol<STD>(M, s) ? 2.5 * M.Rs[s] : 1.5 * M.Rs[s], a);
    return a;
}

// Newton iteration on sum rho_s e_s(T) = rho e, from T0; returns iterations,
// or -1 if maxit was reached.  Stops when |dT| <= tol*T, or when the residual
// is at the rounding level of the energies it is made of (8 eps times
// |rho e| + sum_s |rho_s e0_s|): where the thermal energy is itself that small
// (near-vacuum gas left by the positivity limiter, T of order 1e-10 K) no
// iterate meets a relative test, and T is as accurate as the data allow.
// What bounds it: the FP64 issue of the exponentials.  Each iteration is one
// reciprocal of T, three exponentials and reciprocals (mix_vib) and one
// Newton quotient; the parts linear in T (rho cv without vibration, the
// formation energies) are summed once before the loop.  With the library's
// exp and expm1 (two branches) and the per-species sums inside the loop, the
// indicator with this solve took 55 us on the curved 24^3 N = 4 mesh; now 45.
template <bool STD>
__device__ __forceinline__ int mix_newton_t(const MixC &M, const double *rs, double rhoe_target, double &T,
                                            double tol, int maxit) {
    double floor = fabs(rhoe_target), b = -rhoe_target;
#pragma unroll
    for (int s = 0; s < kNS; ++s) {
        floor = fma(fabs(rs[s]), fabs(M.e0[s]), floor);
        b = fma(rs[s], M.e0[s], b);
    }
    floor *= 8.0 * 2.220446049250313e-16;
    const double a = mix_cv_rigid<STD>(M, rs);
#pragma unroll 1
    for (int it = 1; it <= maxit; ++it) {
        double ev, cv;
        mix_vib<STD>(M, rs, T, ev, cv);
        const double r = fma(a, T, b) + ev;
        // r / fp with a residual correction (the quotient to its last digit)
        const double fp = a + cv, ifp = rcp(fp);
        double dT = r * ifp;
        dT = fma(fma(-fp, dT, r), ifp, dT);
        T -= dT;
        if (fabs(dT) <= tol * fabs(T) || fabs(r) <= floor) return it;
    }
    return -1;
}

__device__ __forceinline__ int mix_newton(const MixC &M, const double *rs, double rhoe_target, double &T, double tol,
                                          int maxit) {
    return M.std_mol ? mix_newton_t<true>(M, rs, rhoe_target, T, tol, maxit)
                     : mix_newton_t<false>(M, rs, rhoe_target, T, tol, maxit);
}

__device__ __forceinline__ double mix_rR(const MixC &M, const double *rs) {
    double r = 0.0;
#pragma unroll
    for (int s = 0; s < kNS; ++s) r = fma(rs[s], M.Rs[s], r);
    return r;
}

// Frozen sound speed sqrt(gamma_f p / rho), gamma_f = 1 + sum rho_s R_s / sum rho_s cv_s.
__device__ __forceinline__ double mix_sound(const MixC &M, const double *rs, double rho, double T) {
    double ev, cv;
    if (M.std_mol) {
        mix_vib<true>(M, rs, T, ev, cv);
        cv += mix_cv_rigid<true>(M, rs);
    } else {
        mix_vib<false>(M, rs, T, ev, cv);
        cv += mix_cv_rigid<false>(M, rs);
    }
    const double rR = mix_rR(M, rs);
    const double g = fma(rR, rcp(cv), 1.0);
    return wave_sqrt(g * rR * T * rcp(rho));
}

// State of a node from its conserved vector (and T for a mixture).
template <int DIM, bool MIX>
// (mixtures: c is the given frozen sound speed when cgiven is not null)
__device__ __forceinline__ void make_state(const double *u, double T, double gamma, const MixC &M,
                                           St<DIM, MIX> &s, const double *cgiven = nullptr) {
    if constexpr (MIX) {
        double rho = 0.0;
#pragma unroll
        for (int k = 0; k < kNS; ++k) {
            s.rs[k] = u[k];
            rho += u[k];
        }
        s.rho = rho;
        const double ir = rcp(rho);
#pragma unroll
        for (int c = 0; c < DIM; ++c) s.v[c] = u[kNS + c] * ir;
        s.rhoE = u[kNS + DIM];
        const double rR = mix_rR(M, s.rs);
        s.p = rR * T;
        s.c = cgiven ? *cgiven : mix_sound(M, s.rs, rho, T);
    } else {
        s.rho = u[0];
        const double ir = rcp(u[0]);
        double v2 = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            s.v[c] = u[1 + c] * ir;
            v2 = fma(s.v[c], s.v[c], v2);
        }
        s.rhoE = u[1 + DIM];
        s.p = (gamma - 1.0) * (s.rhoE - 0.5 * s.rho * v2);
        s.c = wave_sqrt(gamma * s.p * ir);
        s.rs[0] = 0.0;
    }
}

// f(u).n
template <int DIM, bool MIX>
__device__ __forceinline__ void phys_flux(const St<DIM, MIX> &s, const double *n, double *f) {
    const double vn = dotn<DIM>(s.v, n);
    constexpr int off = MIX ? kNS : 1;
    if constexpr (MIX) {
#pragma unroll
        for (int k = 0; k < kNS; ++k) f[k] = s.rs[k] * vn;
    } else {
        f[0] = s.rho * vn;
    }
#pragma unroll
    for (int c = 0; c < DIM; ++c) f[off + c] = s.rho * s.v[c] * vn + s.p * n[c];
    f[off + DIM] = (s.rhoE + s.p) * vn;
}

template <int DIM, bool MIX>
__device__ __forceinline__ void cons_of(const St<DIM, MIX> &s, double *u) {
    constexpr int off = MIX ? kNS : 1;
    if constexpr (MIX) {
#pragma unroll
        for (int k = 0; k < kNS; ++k) u[k] = s.rs[k];
    } else {
        u[0] = s.rho;
    }
#pragma unroll
    for (int c = 0; c < DIM; ++c) u[off + c] = s.rho * s.v[c];
    u[off + DIM] = s.rhoE;
}

// HLL flux with the Davis bounds S_L = min(v_L.n - c_L|n|, v_R.n - c_R|n|),
// S_R = max(v_L.n + c_L|n|, v_R.n + c_R|n|) (scaled n): the upwind physical
// flux when both bounds have one sign, otherwise the flux of the single
// intermediate state that conserves the integral over the wave fan.
template <int DIM, bool MIX>
__device__ __forceinline__ void hll(const St<DIM, MIX> &L, const St<DIM, MIX> &R, const double *n,
                                    double *F) {
    constexpr int NV = (MIX ? kNS : 1) + DIM + 1;
    const double nn = wave_sqrt(dotn<DIM>(n, n));
    const double vL = dotn<DIM>(L.v, n), vR = dotn<DIM>(R.v, n);
    const double sL = fmin(vL - L.c * nn, vR - R.c * nn);
    const double sR = fmax(vL + L.c * nn, vR + R.c * nn);
    if (sL >= 0.0) {
        phys_flux<DIM, MIX>(L, n, F);
    } else if (sR <= 0.0) {
        phys_flux<DIM, MIX>(R, n, F);
    } else {
        double fL[NV], fR[NV], uL[NV], uR[NV];
        phys_flux<DIM, MIX>(L, n, fL);
        phys_flux<DIM, MIX>(R, n, fR);
        cons_of<DIM, MIX>(L, uL);
        cons_of<DIM, MIX>(R, uR);
        const double iw = 1.0 / (sR - sL);
        const double sLR = sL * sR;
#pragma unroll
        for (int k = 0; k < NV; ++k) F[k] = (sR * fL[k] - sL * fR[k] + sLR * (uR[k] - uL[k])) * iw;
    }
}

// HLLC flux, the HLL bounds with Toro's contact speed
// S* = (p_R - p_L + rho_L u_L (S_L - u_L) - rho_R u_R (S_R - u_R))
//      / (rho_L (S_L - u_L) - rho_R (S_R - u_R)) on the unit normal, and the
// star states rho_K (S_K - u_K)/(S_K - S*) (1, v_K + (S* - u_K) n,
// E_K/rho_K + (S* - u_K)(S* + p_K/(rho_K (S_K - u_K)))); scaled by |n|.  For
// a mixture c is the frozen sound speed and the species densities of a star
// state scale like its total density.
template <int DIM, bool MIX>
__device__ __forceinline__ void hllc(const St<DIM, MIX> &L, const St<DIM, MIX> &R, const double *n,
                                     double *F) {
    constexpr int off = MIX ? kNS : 1;
    constexpr int NV = off + DIM + 1;
    const double nn = wave_sqrt(dotn<DIM>(n, n));
    const double inn = rcp(nn);
    double nh[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) nh[c] = n[c] * inn;
    const double uL = dotn<DIM>(L.v, nh), uR = dotn<DIM>(R.v, nh);
    const double sL = fmin(uL - L.c, uR - R.c);
    const double sR = fmax(uL + L.c, uR + R.c);
    const St<DIM, MIX> &K = sL >= 0.0 ? L : R;  // the upwind state when 0 is outside the fan
    if (sL >= 0.0 || sR <= 0.0) {
        phys_flux<DIM, MIX>(K, n, F);
        return;
    }
    const double mL = L.rho * (sL - uL), mR = R.rho * (sR - uR);
    const double ss = (R.p - L.p + mL * uL - mR * uR) / (mL - mR);
    const bool left = ss >= 0.0;
    const St<DIM, MIX> &S = left ? L : R;
    const double sk = left ? sL : sR, uk = left ? uL : uR, mk = left ? mL : mR;
    double f[NV], u[NV], us[NV];
    phys_flux<DIM, MIX>(S, nh, f);
    cons_of<DIM, MIX>(S, u);
    const double fac = mk / (sk - ss);
    if constexpr (MIX) {
#pragma unroll
        for (int k = 0; k < kNS; ++k) us[k] = fac * (S.rs[k] / S.rho);
    } else {
        us[0] = fac;
    }
#pragma unroll
    for (int c = 0; c < DIM; ++c) us[off + c] = fac * (S.v[c] + (ss - uk) * nh[c]);
    us[off + DIM] = fac * (S.rhoE / S.rho + (ss - uk) * (ss + S.p / mk));
#pragma unroll
    for (int k = 0; k < NV; ++k) F[k] = (f[k] + sk * (us[k] - u[k])) * nn;
}

// The standard-DG form as a two-point flux: (f(u_L) + f(u_R)).n / 2.
template <int DIM, bool MIX>
__device__ __forceinline__ void central_state(const St<DIM, MIX> &L, const St<DIM, MIX> &R, const double *n,
                                              double *F) {
    constexpr int NV = (MIX ? kNS : 1) + DIM + 1;
    double fL[NV], fR[NV];
    phys_flux<DIM, MIX>(L, n, fL);
    phys_flux<DIM, MIX>(R, n, fR);
#pragma unroll
    for (int k = 0; k < NV; ++k) F[k] = 0.5 * sum2(fL[k], fR[k]);
}

template <int DIM, bool MIX>
__device__ __forceinline__ void rusanov(const St<DIM, MIX> &L, const St<DIM, MIX> &R,
                                        const double *n, double *F) {
    constexpr int NV = (MIX ? kNS : 1) + DIM + 1;
    const double nn = wave_sqrt(dotn<DIM>(n, n));
    const double lam = fmax(fabs(dotn<DIM>(L.v, n)) + L.c * nn, fabs(dotn<DIM>(R.v, n)) + R.c * nn);
    double fL[NV], fR[NV], uL[NV], uR[NV];
    phys_flux<DIM, MIX>(L, n, fL);
    phys_flux<DIM, MIX>(R, n, fR);
    cons_of<DIM, MIX>(L, uL);
    cons_of<DIM, MIX>(R, uR);
#pragma unroll
    for (int k = 0; k < NV; ++k) F[k] = 0.5 * (fL[k] + fR[k]) - 0.5 * lam * (uR[k] - uL[k]);
}

// Ranocha flux from primitive values (perfect gas).
template <int DIM>
__device__ __forceinline__ void ranocha_prims(double rL, const double *vL, double pL, double bL, double rR,
                                              const double *vR, double pR, double bR, const double *n,
                                              double gm1_inv, double *F) {
    const double rho_hat = ln_mean(rL, rR);
    const double ibeta_hat = inv_ln_mean(bL, bR);
    double vbar[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) vbar[c] = 0.5 * (vL[c] + vR[c]);
    const double pbar = 0.5 * (pL + pR);
    const double q = 0.5 * dotn<DIM>(vL, vR);
    const double frho = rho_hat * dotn<DIM>(vbar, n);
    F[0] = frho;
#pragma unroll
    for (int c = 0; c < DIM; ++c) F[1 + c] = frho * vbar[c] + pbar * n[c];
    F[1 + DIM] = frho * (q + gm1_inv * ibeta_hat) + 0.5 * sum2(pL * dotn<DIM>(vR, n), pR * dotn<DIM>(vL, n));
}

template <int DIM, bool MIX>
__device__ __forceinline__ void ranocha_state(const St<DIM, MIX> &L, const St<DIM, MIX> &R,
                                              const double *n, double gamma, double *F) {
    const double bL = L.rho / L.p, bR = R.rho / R.p;
    ranocha_prims<DIM>(L.rho, L.v, L.p, bL, R.rho, R.v, R.p, bR, n, 1.0 / (gamma - 1.0), F);
}

// Split forms as two-point fluxes with arithmetic means {{a}} = (a_L + a_R)/2.
// FORM 0 Kennedy-Gruber and 1 Pirozzoli: mass flux f = {{rho}}{{v.n}}
// (mixtures: species rows f {{rho_s/rho}}), momentum f {{v}} + {{p}} n,
// energy f {{E/rho}} + {{p}}{{v.n}} (Kennedy-Gruber) or f {{(E + p)/rho}}
// (Pirozzoli).  FORM 2 Morinishi (perfect gas): f = {{rho v}}.n, momentum as
// above, energy f ({{p/((gamma-1) rho)}} + v_L.v_R/2) + {{p v}}.n.
// The perfect gas takes E/rho, (E + p)/rho or p/rho of the nodes from rs[0]
// (pair_quantity: one division per node instead of two per pair).
template <int DIM, int VF>
__device__ __forceinline__ double pair_quantity(double rho, double p, double rhoE) {
    return (VF == 0 ? rho : VF == 2 ? rhoE : VF == 3 ? rhoE + p : p) * rcp(VF == 0 ? p : rho);
}

template <int DIM, bool MIX, int FORM>
__device__ __forceinline__ void split_form_state(const St<DIM, MIX> &L, const St<DIM, MIX> &R,
                                                 const double *n, double gm1_inv, double *F) {
    static_assert(!(MIX && FORM == 2), "Morinishi's form is perfect-gas only");
    constexpr int off = MIX ? kNS : 1;
    double vb[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) vb[c] = 0.5 * (L.v[c] + R.v[c]);
    const double vn = dotn<DIM>(vb, n);
    const double pbar = 0.5 * (L.p + R.p);
    double fm;
    if constexpr (FORM == 2) {
        double mb[DIM];
#pragma unroll
        for (int c = 0; c < DIM; ++c) mb[c] = 0.5 * sum2(L.rho * L.v[c], R.rho * R.v[c]);
        fm = dotn<DIM>(mb, n);
    } else {
        fm = 0.5 * (L.rho + R.rho) * vn;
    }
    double xm;  // mean of the nodal quantity
    if constexpr (MIX) {
        const double iL = rcp(L.rho), iR = rcp(R.rho);
#pragma unroll
        for (int k = 0; k < kNS; ++k) F[k] = fm * (0.5 * sum2(L.rs[k] * iL, R.rs[k] * iR));
        if constexpr (FORM == 1) xm = 0.5 * sum2((L.rhoE + L.p) * iL, (R.rhoE + R.p) * iR);
        else xm = 0.5 * sum2(L.rhoE * iL, R.rhoE * iR);
    } else {
        F[0] = fm;
        xm = 0.5 * (L.rs[0] + R.rs[0]);
    }
#pragma unroll
    for (int c = 0; c < DIM; ++c) F[off + c] = fm * vb[c] + pbar * n[c];
    if constexpr (FORM == 2) {
        double pv[DIM];
#pragma unroll
        for (int c = 0; c < DIM; ++c) pv[c] = 0.5 * sum2(L.p * L.v[c], R.p * R.v[c]);
        F[off + DIM] = fm * (xm * gm1_inv + 0.5 * dotn<DIM>(L.v, R.v)) + dotn<DIM>(pv, n);
    } else if constexpr (FORM == 1) {
        F[off + DIM] = fm * xm;
    } else {
        F[off + DIM] = fm * xm + pbar * vn;
    }
}

// What the entropy-conservative mixture flux takes of a node: beta = 1/T, the
// gas constant density sum_s rho_s R_s and, per molecule among the first
// three species, D = exp(-theta beta / 2) - 1 (a molecule elsewhere in the
// species table takes its exponentials in the flux).  D and not the exponential
// itself: 1 - exp(-theta beta) = -D (2 + D) keeps its digits in hot gas, where
// the square of the rounded exponential subtracted from 1 loses them (relative
// error of the energy mean, rms, at 20,000 K 1.1e-16 against 1.4e-16, at 1e6 K
// against 4e-15), and in cold gas, where only 1 + D is rounded at the size of 1,
// the vibrational part is as small (1.2e-16 from 100 K on).  It costs two
// instructions per molecule and node: the curved 16^3 right-hand side takes 135.7
// us, with the exponentials 134.5.
constexpr int kEcMol = 3;
template <int DIM>
struct EcNode {
    double rs[kNS], v[DIM], rR, beta, D[kEcMol];
};

__device__ __forceinline__ double expm1_neg_half(double th, double beta) {
    int n;
    const double p = expm1_reduced(-0.5 * th * beta, n);
    const double s = ldexp(1.0, n);
    return fma(s, p, s - 1.0);
}

template <int DIM>
__device__ __forceinline__ void ec_node(const double *rs, const double *v, double T, const MixC &M, EcNode<DIM> &e) {
#pragma unroll
    for (int k = 0; k < kNS; ++k) e.rs[k] = rs[k];
#pragma unroll
    for (int c = 0; c < DIM; ++c) e.v[c] = v[c];
    e.rR = mix_rR(M, rs);
    e.beta = rcp(T);
#pragma unroll
    for (int k = 0; k < kEcMol; ++k) e.D[k] = expm1_neg_half(M.thv[k], e.beta);
}

// exp(-theta bbar) sinh(z)/z, z = theta (bR - bL)/2, from the two exponentials
// exp(-theta beta / 2): the series of sinh(z)/z to z^18 (remainder < 3e-20) for
// |z| < 1, else the difference of the squares (a ratio above e^2, no
// cancellation).
__device__ __forceinline__ double exp_sinhc(double th, double db, double EL, double ER) {
    const double z = 0.5 * th * db, y = z * z;
    double r = poly_start(y, 1.0 / 121645100408832000.0, 1.0 / 355687428096000.0);
    r = fma_kv(r, y, 1.0 / 1307674368000.0);
    r = fma_kv(r, y, 1.0 / 6227020800.0);
    r = fma_kv(r, y, 1.0 / 39916800.0);
    r = fma_kv(r, y, 1.0 / 362880.0);
    r = fma_kv(r, y, 1.0 / 5040.0);
    r = fma_kv(r, y, 1.0 / 120.0);
    r = fma_kv(r, y, 1.0 / 6.0);
    double s = EL * ER * fma(y, r, 1.0);
    if (fabs(z) >= 1.0) s = fma(EL, EL, -ER * ER) * rcp(th * db);
    return s;
}

// Entropy-conservative flux of the RRHO mixture (Tadmor's condition with
// the mixture entropy -sum rho_s s_s; beta = 1/T = sum rho_s R_s / p):
// species fluxes rho_s^ln {{v}}.n (0 where a density is 0, the limit),
// momentum F_rho {{v}} + p~ n with p~ = {{sum rho_s R_s}}/{{beta}}, energy
// sum_s e^_s F_s + F_rho (|{{v}}|^2 - {{|v|^2}}/2) + p~ {{v}}.n, with the
// energy means e^_s = e0_s + c_s / beta^ln (c_s = 3/2 R_s, 5/2 R_s for
// molecules) + R_s theta_s exp(-theta_s {{beta}}) sinhc(theta_s [[beta]]/2)
// / ln-mean(1 - exp(-theta_s beta)) for molecules.
//
// What bounds it: FP64 issue.  A pair needs nine logarithmic means and three
// exp-sinhc terms; with every exponential (three per molecule) evaluated per
// pair by the library and the means in three branches, k_rhs on the curved
// 16^3 N = 4 mesh took 184 us.  A node meets 12 partners, so its exponentials
// are evaluated once (EcNode) and the pair multiplies them: about 500 vector
// instructions per pair instead of 1,500 (the far branch of a trace species'
// mean runs in two thirds of the waves there), k_rhs 118 us.
template <int DIM>
__device__ __forceinline__ void ec_mixture_pair(const EcNode<DIM> &L, const EcNode<DIM> &R, const double *n,
                                                const MixC &M, double *F) {
    const double db = R.beta - L.beta;
    const double iblog = inv_ln_mean_wide(L.beta, R.beta);
    double vb[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) vb[c] = 0.5 * (L.v[c] + R.v[c]);
    const double vn = dotn<DIM>(vb, n);
    const double pt = (L.rR + R.rR) * rcp(L.beta + R.beta);
    double sm = 0.0, en = 0.0;
#pragma unroll
    for (int k = 0; k < kNS; ++k) {
        const double m = ln_mean_wide(L.rs[k], R.rs[k]);
        F[k] = m * vn;
        sm += m;
        double eh = M.e0[k];
        if (M.mol[k]) {
            const double th = M.thv[k];
            const double DL = k < kEcMol ? L.D[k < kEcMol ? k : 0] : expm1_neg_half(th, L.beta);
            const double DR = k < kEcMol ? R.D[k < kEcMol ? k : 0] : expm1_neg_half(th, R.beta);
            const double t = exp_sinhc(th, db, 1.0 + DL, 1.0 + DR) * inv_ln_mean_wide(-DL * (2.0 + DL), -DR * (2.0 + DR));
            eh = fma(M.Rs[k], fma(th, t, 2.5 * iblog), eh);
        } else {
            eh = fma(M.Rs[k], 1.5 * iblog, eh);
        }
        en = fma(eh, m, en);
        __builtin_amdgcn_sched_barrier(0);
    }
    const double frho = sm * vn;
#pragma unroll
    for (int c = 0; c < DIM; ++c) F[kNS + c] = fma(frho, vb[c], pt * n[c]);
    const double k2 = dotn<DIM>(vb, vb) - 0.25 * (dotn<DIM>(L.v, L.v) + dotn<DIM>(R.v, R.v));
    F[kNS + DIM] = vn * (fma(sm, k2, en) + pt);
}

// the same from two node states (faces)
template <int DIM>
__device__ __forceinline__ void ec_mixture_state(const St<DIM, true> &L, const St<DIM, true> &R, const double *n,
                                                 const MixC &M, double *F) {
    EcNode<DIM> A, B;
    ec_node<DIM>(L.rs, L.v, L.p * rcp(mix_rR(M, L.rs)), M, A);
    ec_node<DIM>(R.rs, R.v, R.p * rcp(mix_rR(M, R.rs)), M, B);
    ec_mixture_pair<DIM>(A, B, n, M, F);
}

// Ducros split-form flux: {{rho_s}} {{v}}.n, {{m}} {{v}}.n + {{p}} n, ({{rhoE}} + {{p}}) {{v}}.n
template <int DIM, bool MIX>
__device__ __forceinline__ void ducros_state(const St<DIM, MIX> &L, const St<DIM, MIX> &R,
                                             const double *n, double *F) {
    double vb[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) vb[c] = 0.5 * (L.v[c] + R.v[c]);
    const double vn = dotn<DIM>(vb, n);
    const double pbar = 0.5 * (L.p + R.p);
    constexpr int off = MIX ? kNS : 1;
    if constexpr (MIX) {
#pragma unroll
        for (int k = 0; k < kNS; ++k) F[k] = 0.5 * (L.rs[k] + R.rs[k]) * vn;
    } else {
        F[0] = 0.5 * (L.rho + R.rho) * vn;
    }
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        const double mbar = 0.5 * sum2(L.rho * L.v[c], R.rho * R.v[c]);
        F[off + c] = mbar * vn + pbar * n[c];
    }
    F[off + DIM] = (0.5 * (L.rhoE + R.rhoE) + pbar) * vn;
}

}  // namespace dgx
