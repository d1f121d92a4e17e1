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
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <iostream>
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
    return 1;
}
