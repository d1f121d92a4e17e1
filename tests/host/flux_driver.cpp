// CPU driver of the device-side means and two-point fluxes (csrc/physics.h) for
// the tests.  physics.h is included from a copy without its HIP include and its
// empty asm statements (register hints), and the hardware's reciprocal and
// mantissa instructions are given here.  Reads a command and numbers on stdin,
// prints hexadecimal doubles.
//
//   means   n, then n lines "x y": ln_mean, inv_ln_mean, ln_mean_wide,
//           inv_ln_mean_wide
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
    return 1;
}
