// CPU driver of the device-side means and two-point fluxes (csrc/physics.h) for
// the tests.  physics.h is included from a copy without its HIP include and its
// empty asm statements (register hints), and the hardware's reciprocal and
// mantissa instructions are given here.  Reads a command and numbers on stdin,
// prints hexadecimal doubles.
//
//   means   n, then n lines "x y": ln_mean, inv_ln_mean, ln_mean_wide,
//           inv_ln_mean_wide
//   ec      n, then n lines "theta R TL TR": the energy row of the entropy-
//           conservative mixture flux of a gas of one molecule, density 1,
//           formation energy 0, at unit velocity through a unit face
//   swap    n: the two-point fluxes of n random pairs of states, the pair taken
//           both ways; prints per flux how many differ in some bit: perfect gas
//           Ranocha, Ducros, Kennedy-Gruber, Pirozzoli, central, Morinishi,
//           then the mixture's Ducros, Kennedy-Gruber, Pirozzoli, central
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <iostream>
#include <random>
#include <string>

using std::max;
using std::min;

#define __device__
#define __host__
#define __forceinline__ inline
static double driver_mant(double x) {
    int e;
    return std::frexp(x, &e);
}
static int driver_exp(double x) {
    int e;
    std::frexp(x, &e);
    return e;
}
static long long __double_as_longlong(double x) {
    long long i;
    std::memcpy(&i, &x, sizeof(i));
    return i;
}
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_rsq(x) (1.0 / std::sqrt(x))
#define __builtin_amdgcn_frexp_mant(x) driver_mant(x)
#define __builtin_amdgcn_frexp_exp(x) driver_exp(x)
#define __builtin_amdgcn_sched_barrier(x)

#include "physics.h"

using namespace dgx;

static double number() {
    std::string s;
    std::cin >> s;
    return std::strtod(s.c_str(), nullptr);
}

// (not inlined: the two orders must not share their products)
template <bool MIX, int VF>
__attribute__((noinline)) static void pair_flux(const St<3, MIX> &A, const St<3, MIX> &B, const double *n, double *F) {
    const double gm1_inv = 1.0 / 0.4;
    if constexpr (VF == 0) ranocha_prims<3>(A.rho, A.v, A.p, A.rs[0], B.rho, B.v, B.p, B.rs[0], n, gm1_inv, F);
    else if constexpr (VF == 1) ducros_state<3, MIX>(A, B, n, F);
    else if constexpr (VF == 4) central_state<3, MIX>(A, B, n, F);
    else split_form_state<3, MIX, VF == 2 ? 0 : VF == 3 ? 1 : 2>(A, B, n, gm1_inv, F);
}

template <bool MIX, int VF>
static int unequal_swaps(int n) {
    std::mt19937_64 rng(6);
    std::uniform_real_distribution<double> U(-1.0, 1.0);
    constexpr int NV = (MIX ? kNS : 1) + 4;
    int bad = 0;
    for (int i = 0; i < n; ++i) {
        St<3, MIX> s[2];
        for (auto &x : s) {
            x.rho = 0.0;
            if constexpr (MIX) {
                for (double &r : x.rs) x.rho += r = 1.1 + U(rng);
            } else {
                x.rho = 1.1 + U(rng);
            }
            for (double &v : x.v) v = U(rng);
            x.p = 1.1 + U(rng);
            x.rhoE = 4.0 + U(rng);
            x.c = 1.0;
            if constexpr (!MIX && VF != 1 && VF != 4) x.rs[0] = pair_quantity<3, VF>(x.rho, x.p, x.rhoE);
        }
        const double nrm[3] = {U(rng), U(rng), U(rng)};
        double F[NV], G[NV];
        pair_flux<MIX, VF>(s[0], s[1], nrm, F);
        pair_flux<MIX, VF>(s[1], s[0], nrm, G);
        bad += std::memcmp(F, G, sizeof(F)) != 0;
    }
    return bad;
}

int main() {
    std::string cmd;
    int n;
    std::cin >> cmd >> n;
    if (cmd == "means") {
        for (int i = 0; i < n; ++i) {
            const double x = number(), y = number();
            std::printf("%a %a %a %a\n", ln_mean(x, y), inv_ln_mean(x, y), ln_mean_wide(x, y), inv_ln_mean_wide(x, y));
        }
        return 0;
    }
    if (cmd == "ec") {
        for (int i = 0; i < n; ++i) {
            MixC M{};
            M.thv[0] = number();
            M.Rs[0] = number();
            M.mol[0] = 1;
            const double TL = number(), TR = number();
            const double rs[kNS] = {1.0}, v[3] = {1.0, 0.0, 0.0};
            EcNode<3> A, B;
            ec_node<3>(rs, v, TL, M, A);
            ec_node<3>(rs, v, TR, M, B);
            double F[kNS + 4];
            ec_mixture_pair<3>(A, B, v, M, F);
            std::printf("%a\n", F[kNS + 3]);
        }
        return 0;
    }
    if (cmd == "swap") {
        for (int bad : {unequal_swaps<false, 0>(n), unequal_swaps<false, 1>(n), unequal_swaps<false, 2>(n),
                        unequal_swaps<false, 3>(n), unequal_swaps<false, 4>(n), unequal_swaps<false, 5>(n),
                        unequal_swaps<true, 1>(n), unequal_swaps<true, 2>(n), unequal_swaps<true, 3>(n),
                        unequal_swaps<true, 4>(n)})
            std::printf("%d\n", bad);
        return 0;
    }
    return 1;
}
