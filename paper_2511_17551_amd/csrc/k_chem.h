// Per-node stiff chemistry: backward-Euler steps of the species sources
// (Governing Equations, Eq. source_term; Appendix, Chemical Kinetics) with
// the transport split off.  Density, momentum and total energy stay fixed,
// hence so does rho e, and one step over h from rho_s^a solves
//
//   G(rho_s) = rho_s - rho_s^a - h * omega_s(rho_s, T(rho_s, rho e)) = 0.
//
// Newton's method with the analytic Jacobian along the fixed-energy manifold,
//   d omega_s / d rho_j = W_s sum_r dnu_rs [ (dR_r/dc_j) / W_j
//                                            + (dR_r/dT) dT/drho_j ],
//   dT/drho_j = -e_j(T) / sum_k rho_k cv_k(T),
// where dR_r/dT uses d ln k_f/dT = (b + theta_a/T)/T and the van 't Hoff form
// d ln K_c/dT = -sum_s dnu_s/T + sum_s dnu_s h_s / (R_s T^2), h_s = e_s + R_s T
// (the Gibbs-Helmholtz relation of the Gibbs energies the rates use).  Each
// iterate's temperature comes from the T(e) Newton solve warm-started at the
// previous one.  The step is limited so that densities stay non-negative and
// the thermal energy rho e - sum_s rho_s e0_s stays positive; the iteration
// stops when the full Newton step is below tol * rho.
//
// Substeps.  A growing mode (atom-impact dissociation grows [X] at a rate
// k [X2]) makes I - h d omega/d rho singular as h times its growth rate
// reaches 1; past that the root near rho^a is gone, the Newton step points
// out of the admissible set and the positivity limit cuts it to nothing.  The
// iteration has failed when that limit leaves less than kChemStall of the
// step on two consecutive iterations (or after maxit iterations); the node
// then covers dt with substeps dt / 2^k: a failed substep is retried at half
// the size, and after a successful one the node goes back to the next larger
// size when its position is a multiple of it.  Positions are integers in
// units of dt / 2^kChemKmax; failing at the smallest size is
// non-convergence.
#pragma once

#include "physics.h"

namespace dgx {

// The reaction data to be read where it stands: through a pointer that the
// compiler cannot see through, or it hoists some forty constants out of the
// Newton and group loops and holds them in lanes of spilled registers (fifty
// lane reads per group and 69 spilled VGPRs, against scalar loads that hit).
using KinConst = const __attribute__((address_space(4))) KinC;
__device__ __forceinline__ KinConst *kin_here(const KinC &K) {
    uint64_t p = reinterpret_cast<uint64_t>(&K);
    asm volatile("" : "+s"(p));
    return (KinConst *)p;
}

// Species sources w_s (kg m^-3 s^-1) and their Jacobian dw[s][j] =
// d w_s / d rho_j along the fixed-energy manifold, at the temperature T of
// the composition rs: the mechanisms of grouped form (KinGroups) with the
// molecules first.
//
// What bounds it: the dependency chains and issue of one node's arithmetic (a
// thread per node, two waves per SIMD).  Reaction by reaction, as in
// chem_sources below, most of the time went into uniform branches over the
// stoichiometric coefficients (about 80 per reaction) and two library
// exponentials per reaction.  Here a group evaluates ln K_c and its factor
// products once; k_b = k_f / K_c comes from the two reduced exponentials and
// the sum of their binary exponents, which neither under- nor overflows
// before the final scaling (near 0 K, where the exponents leave the range of
// an int, from the exponential of ln k_f - ln K_c); the factors are gathered
// and their derivatives scattered with one-hot coefficients (exact); and the
// temperature part of the Jacobian is one outer product at the end.  k_chem on the 64 x 128
// cylinder (131,072 nodes, hot state): 184 us reaction by reaction, 78 us
// grouped (74 with the data read in place, the T(e) solve of 6 us included),
// so the grouped form is taken wherever it exists.
__device__ __forceinline__ void chem_sources_grouped(const KinC &K, const double *rs, double T, double *w,
                                                     double (*dw)[kNS]) {
    KinConst *K0 = kin_here(K);
    const double lnT = log(T);
    const double iT = rcp(T);
    double gRT[kNS], dgRT[kNS], conc[kNS], dTdr[kNS], wT[kNS];
    double rhocv = 0.0;
#pragma unroll
    for (int s = 0; s < kNS; ++s) {
        const bool mol = s < 3;
        const double h = K0->th0[s] * iT;            // e0_s / (R_s T)
        double ert = (mol ? 2.5 : 1.5) + h;        // e_s / (R_s T)
        double cvr = mol ? 2.5 : 1.5;              // cv_s / R_s
        double g = K0->gconst[s] - (mol ? 3.5 : 2.5) * lnT + h;
        if (mol) {
            const double x = K0->thv[s] * iT;
            double em, om;  // e^-x, 1 - e^-x
            exp_pair(x, em, om);
            const double io = rcp(om);
            const double xq = x * em * io;
            ert += xq;
            cvr = fma(xq, x * io, cvr);
            g += log(om);
        }
        gRT[s] = g;                      // g_s / (R_s T)
        dgRT[s] = -(ert + 1.0) * iT;     // its T-derivative -h_s / (R_s T^2)
        dTdr[s] = -K0->Rs[s] * T * ert;    // -e_s, scaled below
        rhocv = fma(rs[s] * K0->Rs[s], cvr, rhocv);
        conc[s] = rs[s] * K0->iW[s];
        w[s] = 0.0;
        wT[s] = 0.0;
#pragma unroll
        for (int j = 0; j < kNS; ++j) dw[s][j] = 0.0;
    }
    const double lnpr = K0->lnpref_Ru - lnT;
#pragma unroll 1
    for (int g = 0; g < K0->G.ng; ++g) {
        KinConst *Kg = kin_here(K);
        const __attribute__((address_space(4))) KinGroups &G = Kg->G;
        double mlnK = -G.dn_sum[g] * lnpr;  // -ln K_c
        double dlnK = -G.dn_sum[g] * iT;    // d ln K_c / dT
#pragma unroll
        for (int s = 0; s < kNS; ++s) {
            mlnK = fma(G.dn[g][s], gRT[s], mlnK);
            dlnK = fma(-G.dn[g][s], dgRT[s], dlnK);
        }
        int nK;
        const double mK = 1.0 + expm1_reduced(mlnK, nK);
        const bool in_range = fabs(mlnK) < 4e8;
        double f[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[i] = G.one[g][i];
#pragma unroll
            for (int s = 0; s < kNS; ++s) f[i] = fma(G.sel[g][i][s], conc[s], f[i]);
        }
        const double F = f[0] * f[1], B = f[2] * f[3];
        // sums over the partners: k_f c_M, k_b c_M and their T-derivatives
        double Sf = 0.0, Sb = 0.0, Tf = 0.0, Tb = 0.0, val[kNS];
#pragma unroll
        for (int j = 0; j < kNS; ++j) val[j] = 0.0;
        const int mask = G.mask[g];
        auto partner = [&](int m, double c) {
            const double lnkf = fma(G.b[g][m], lnT, G.lnA[g][m]) - G.tha[g][m] * iT;
            const double dl = fma(G.tha[g][m], iT, G.b[g][m]) * iT;
            int n;
            const double mf = 1.0 + expm1_reduced(lnkf, n);
            const double kf = ldexp(mf, n);
            double kb = ldexp(mf * mK, n + nK);
            if (!in_range) {
                const double mb = 1.0 + expm1_reduced(lnkf + mlnK, n);
                kb = ldexp(mb, n);
            }
            const double cf = kf * c, cb = kb * c;
            Sf += cf;
            Sb += cb;
            Tf = fma(cf, dl, Tf);
            Tb = fma(cb, dl - dlnK, Tb);
            if (m < kNS) val[m] = kf * F - kb * B;
        };
#pragma unroll
        for (int m = 0; m < kNS; ++m)
            if (mask >> m & 1) partner(m, conc[m]);
        if (mask >> kNS & 1) partner(kNS, 1.0);
        const double R = Sf * F - Sb * B;
#pragma unroll
        for (int s = 0; s < kNS; ++s) w[s] = fma(G.wdn[g][s], R, w[s]);
        const double dRdT = Tf * F - Tb * B;
        const double d0 = Sf * f[1], d1 = Sf * f[0], d2 = -Sb * f[3], d3 = -Sb * f[2];
#pragma unroll
        for (int j = 0; j < kNS; ++j) {
            double v = fma(G.sel[g][0][j], d0, val[j]);
            v = fma(G.sel[g][1][j], d1, v);
            v = fma(G.sel[g][2][j], d2, v);
            v = fma(G.sel[g][3][j], d3, v) * Kg->iW[j];  // dR / d rho_j at fixed T
#pragma unroll
            for (int s = 0; s < kNS; ++s) dw[s][j] = fma(G.wdn[g][s], v, dw[s][j]);
        }
#pragma unroll
        for (int s = 0; s < kNS; ++s) wT[s] = fma(G.wdn[g][s], dRdT, wT[s]);
    }
    const double irc = rcp(rhocv);
#pragma unroll
    for (int j = 0; j < kNS; ++j) {
        const double dT = dTdr[j] * irc;
#pragma unroll
        for (int s = 0; s < kNS; ++s) dw[s][j] = fma(wT[s], dT, dw[s][j]);
    }
}

// The same for any mechanism, reaction by reaction.
__device__ __forceinline__ void chem_sources(const KinC &K, const MixC &M, const double *rs, double T, double *w,
                                             double (*dw)[kNS]) {
    const double lnT = log(T);
    const double iT = rcp(T);
    double gRT[kNS], dgRT[kNS], conc[kNS], es[kNS];
    double rhocv = 0.0;
#pragma unroll
    for (int s = 0; s < kNS; ++s) {
        double e = 1.5 * M.Rs[s] * T + M.e0[s];
        double cv = 1.5 * M.Rs[s];
        double g = K.gconst[s] - 2.5 * lnT + M.e0[s] * iT / M.Rs[s];
        if (M.mol[s]) {
            const double x = M.thv[s] * iT;
            double em, om;  // e^-x, 1 - e^-x
            exp_pair(x, em, om);
            const double q = em * rcp(om);
            e += M.Rs[s] * T + M.Rs[s] * M.thv[s] * q;
            cv += M.Rs[s] + M.Rs[s] * x * x * q * rcp(om);
            g += -lnT + log(om);
        }
        es[s] = e;
        rhocv = fma(rs[s], cv, rhocv);
        gRT[s] = g;                                    // g_s / (R_s T)
        dgRT[s] = -(e + M.Rs[s] * T) * iT * iT / M.Rs[s];  // d(g_s/(R_s T))/dT
        conc[s] = rs[s] / K.W[s];
        w[s] = 0.0;
#pragma unroll
        for (int j = 0; j < kNS; ++j) dw[s][j] = 0.0;
    }
    const double irc = rcp(rhocv);
    double dTdr[kNS];
#pragma unroll
    for (int j = 0; j < kNS; ++j) dTdr[j] = -es[j] * irc;
    const double lnpr = K.lnpref_Ru - lnT;
    for (int r = 0; r < K.nr; ++r) {
        double lnK = K.dnu_sum[r] * lnpr;
        double dlnK = -K.dnu_sum[r] * iT;
        double fw = 1.0, bw = 1.0;
        double dfw[kNS], dbw[kNS];
#pragma unroll
        for (int j = 0; j < kNS; ++j) {
            const int nu = K.nu[r][j], nup = K.nup[r][j];
            lnK -= (double)(nup - nu) * gRT[j];
            dlnK -= (double)(nup - nu) * dgRT[j];
            for (int q = 0; q < nu; ++q) fw *= conc[j];
            for (int q = 0; q < nup; ++q) bw *= conc[j];
        }
        // d(prod_k c_k^nu_k)/dc_j = nu_j c_j^(nu_j - 1) prod_{k != j} c_k^nu_k
#pragma unroll
        for (int j = 0; j < kNS; ++j) {
            double pf = 0.0, pb = 0.0;
            const int nuj = K.nu[r][j], nupj = K.nup[r][j];
            if (nuj > 0) {
                pf = (double)nuj;
                for (int q = 1; q < nuj; ++q) pf *= conc[j];
#pragma unroll
                for (int k = 0; k < kNS; ++k)
                    if (k != j)
                        for (int q = 0; q < K.nu[r][k]; ++q) pf *= conc[k];
            }
            if (nupj > 0) {
                pb = (double)nupj;
                for (int q = 1; q < nupj; ++q) pb *= conc[j];
#pragma unroll
                for (int k = 0; k < kNS; ++k)
                    if (k != j)
                        for (int q = 0; q < K.nup[r][k]; ++q) pb *= conc[k];
            }
            dfw[j] = pf;
            dbw[j] = pb;
        }
        const double lnkf = fma(K.b[r], lnT, K.lnA[r]) - K.tha[r] * iT;
        const double kf = exp(lnkf);
        const double kb = exp(lnkf - lnK);  // k_f / K_c without the underflow of both at low T
        const double dlnkf = (K.b[r] + K.tha[r] * iT) * iT;
        const double R = kf * fw - kb * bw;
        const double dRdT = kf * fw * dlnkf - kb * bw * (dlnkf - dlnK);
        double dRdr[kNS];
#pragma unroll
        for (int j = 0; j < kNS; ++j) dRdr[j] = (kf * dfw[j] - kb * dbw[j]) / K.W[j] + dRdT * dTdr[j];
#pragma unroll
        for (int s = 0; s < kNS; ++s) {
            const int dn = K.nup[r][s] - K.nu[r][s];
            if (dn != 0) {
                const double c = K.W[s] * (double)dn;
                w[s] = fma(c, R, w[s]);
#pragma unroll
                for (int j = 0; j < kNS; ++j) dw[s][j] = fma(c, dRdr[j], dw[s][j]);
            }
        }
    }
}

// x = A^{-1} b for the 5x5 system (Gaussian elimination, partial pivoting;
// row exchanges by selects so that the arrays stay in registers).
__device__ __forceinline__ void solve5(double (*A)[kNS], double *b, double *x) {
    double ip[kNS];  // 1 / pivot
#pragma unroll
    for (int c = 0; c < kNS; ++c) {
        // pivot: the largest |A[k][c]|, k >= c, swapped into row c
        double best = fabs(A[c][c]);
        int piv = c;
#pragma unroll
        for (int k = c + 1; k < kNS; ++k)
            if (fabs(A[k][c]) > best) {
                best = fabs(A[k][c]);
                piv = k;
            }
#pragma unroll
        for (int k = c + 1; k < kNS; ++k) {
            const bool sw = (k == piv);
#pragma unroll
            for (int j = c; j < kNS; ++j) {
                const double t = A[c][j];
                A[c][j] = sw ? A[k][j] : A[c][j];
                A[k][j] = sw ? t : A[k][j];
            }
            const double t = b[c];
            b[c] = sw ? b[k] : b[c];
            b[k] = sw ? t : b[k];
        }
        ip[c] = rcp(A[c][c]);
#pragma unroll
        for (int k = c + 1; k < kNS; ++k) {
            const double f = A[k][c] * ip[c];
#pragma unroll
            for (int j = c + 1; j < kNS; ++j) A[k][j] = fma(-f, A[c][j], A[k][j]);
            b[k] = fma(-f, b[c], b[k]);
        }
    }
#pragma unroll
    for (int c = kNS - 1; c >= 0; --c) {
        double s = b[c];
#pragma unroll
        for (int j = c + 1; j < kNS; ++j) s = fma(-A[c][j], x[j], s);
        x[c] = s * ip[c];
    }
}

constexpr int kChemKmax = 20;        // smallest substep dt / 2^20
constexpr double kChemStall = 1e-3;  // a step cut below this fraction twice in a row has failed

// Damped Newton for one backward-Euler step over h from ra into rs.  Tn: the
// temperature of ra on entry, of rs on a converged exit.  Adds the
// iterations to it; returns false if the iteration failed.
template <bool GRP, bool STD>
__device__ __forceinline__ bool chem_newton(const KinC &K, const MixC &M, const double *ra, double *rs, double rho,
                                            double rhoe, double h, double &Tn, double tol, int maxit, double ttol,
                                            int tmaxit, int &it) {
#pragma unroll
    for (int s = 0; s < kNS; ++s) rs[s] = ra[s];
    auto solve_T = [&]() { return mix_newton_t<STD>(M, rs, rhoe, Tn, ttol, tmaxit); };
    int low = 0;
    for (int k = 0; k < maxit; ++k) {
        ++it;
        if (solve_T() < 0 || !(Tn > 0.0)) return false;
        double w[kNS], A[kNS][kNS], G[kNS], d[kNS];
        if constexpr (GRP) chem_sources_grouped(K, rs, Tn, w, A);
        else chem_sources(K, M, rs, Tn, w, A);
#pragma unroll
        for (int s = 0; s < kNS; ++s) {
            G[s] = -(rs[s] - ra[s] - h * w[s]);
#pragma unroll
            for (int j = 0; j < kNS; ++j) A[s][j] = (s == j ? 1.0 : 0.0) - h * A[s][j];
        }
        solve5(A, G, d);
        // step limits: rho_s >= 0 and a positive thermal energy
        double theta = 1.0, thermal = rhoe, de0 = 0.0, dmax = 0.0;
#pragma unroll
        for (int s = 0; s < kNS; ++s) {
            if (rs[s] + d[s] < 0.0) theta = fmin(theta, -0.9 * rs[s] / d[s]);
            thermal -= rs[s] * M.e0[s];
            de0 = fma(d[s], M.e0[s], de0);
            dmax = fmax(dmax, fabs(d[s]));
        }
        if (de0 > 0.0) theta = fmin(theta, 0.9 * thermal / de0);
#pragma unroll
        for (int s = 0; s < kNS; ++s) rs[s] = fma(theta, d[s], rs[s]);
        if (!(dmax == dmax)) return false;
        if (dmax <= tol * rho) return solve_T() >= 0;
        low = theta < kChemStall ? low + 1 : 0;
        if (low >= 2) return false;
    }
    return false;
}

// Chemistry over dt per node, in place on the species rows of u
// ([nvar][count], species first).  GRP: the grouped rates.  STD: the molecules
// are the first three species (GRP: always); known here, or the two forms of
// the T(e) solve stand side by side and spill (other flags, 131,072 nodes: 2717
// us, now 2197).  Two waves per SIMD: the Newton state, the 5x5 Jacobian and the
// rate terms need about 280 registers, and one wave per SIMD leaves the long
// dependency chains (T solve, rates, elimination) unhidden: two were 1.45x
// faster for the general rates on the 131,072-node cylinder.  No form spills
// VGPRs at this bound.  T holds the incoming state's temperature on entry and
// the new one on exit.  GRP: on entry a warm start, from which (or from T0
// where it is no positive number or fails) the incoming temperature is solved
// for here: as k_thermo before this kernel that took 6 of 80 us on the
// cylinder.  The general rates keep the two launches (the solve's registers
// cost them more: 394 -> 399 us a Strang step).  iters (optional) the Newton
// iterations summed over the substeps, -1 if the node did not converge;
// subs (optional) the number of substeps.
template <int DIM, bool GRP, bool STD>
__global__ void __launch_bounds__(256, 2) k_chem(double *__restrict__ u, int64_t count, double dt, const KinC *kin,
                                              MixC M, double *__restrict__ T, double T0, double ntol, int nmaxit,
                                              double tol, int maxit, double ttol, int tmaxit,
                                              int *__restrict__ iters, int *__restrict__ subs, unsigned *flags) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const KinC &K = *kin;
    double ra[kNS];
    double rho = 0.0;
#pragma unroll
    for (int s = 0; s < kNS; ++s) {
        ra[s] = u[s * count + i];
        rho += ra[s];
    }
    double m2 = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        const double m = u[(kNS + c) * count + i];
        m2 = fma(m, m, m2);
    }
    const double rhoe = u[(kNS + DIM) * count + i] - 0.5 * m2 / rho;
    double Ta = T[i];
    if constexpr (GRP) {
        // (the steps of node_temperature_state)
        if (!(Ta > 0.0) || !isfinite(Ta)) Ta = T0;
        bool found = false;
#pragma unroll 1
        for (int a = 0; a < 2 && !found; ++a) {
            if (a) Ta = T0;
            const int n = mix_newton_t<STD>(M, ra, rhoe, Ta, ntol, nmaxit);
            found = n >= 0 && isfinite(Ta) && Ta > 0.0;
        }
        if (!found) atomicOr(flags, FLAG_NOCONV);
    }
    constexpr int unit = 1 << kChemKmax;
    int pos = 0, lev = 0, it = 0, nsub = 0;
    bool conv = true;
    while (pos < unit) {
        if (lev > kChemKmax) {
            conv = false;
            break;
        }
        double rs[kNS];
        double Tn = Ta;
        if (chem_newton<GRP, STD>(K, M, ra, rs, rho, rhoe, ldexp(dt, -lev), Tn, tol, maxit, ttol, tmaxit, it)) {
#pragma unroll
            for (int s = 0; s < kNS; ++s) ra[s] = rs[s];
            Ta = Tn;
            pos += unit >> lev;
            ++nsub;
            if (lev > 0 && (pos & ((unit >> (lev - 1)) - 1)) == 0) --lev;
        } else {
            ++lev;
        }
    }
#pragma unroll
    for (int s = 0; s < kNS; ++s) u[s * count + i] = ra[s];
    T[i] = Ta;
    if (iters) iters[i] = conv ? it : -1;
    if (subs) subs[i] = nsub;
    if (!conv) atomicOr(flags, FLAG_NOCONV);
}

}  // namespace dgx
