"""The device-side means and two-point fluxes (csrc/physics.h), built here with
clang++ into a CPU driver (tests/host/flux_driver.cpp): the arithmetic as it
stands, with the contraction rules of the HIP build.

* Logarithmic means against extended precision over ratios from 1 to 1e12, and
  at their edges: two equal values give that value, also negative ones, a zero
  gives zero (the mean) and values of opposite sign give no number.
* The energy row of the entropy-conservative mixture flux of a molecule against
  extended precision from 100 K to 1e6 K (where 1 - exp(-theta/T) is 3e-3).
* The other two-point fluxes are bitwise the same for a pair taken either way
  (at N = 3 both nodes evaluate a pair, each with its own state first).
"""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2511_17551_amd", "csrc")
CLANG = shutil.which("amdclang++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("clang++ not available")
    d = tmp_path_factory.mktemp("fluxdrv")
    for name in ("physics.h", "dgx_internal.h"):
        with open(os.path.join(CSRC, name)) as f:
            text = f.read().replace("#include <hip/hip_runtime.h>", "")
        (d / name).write_text(re.sub(r"\basm\b[^;]*;", ";", text))
    exe = str(d / "flux_driver")
    subprocess.run([CLANG, "-O2", "-std=c++17", "-mfma", "-ffp-contract=fast-honor-pragmas", "-Wno-unknown-pragmas",
                    "-I", str(d), os.path.join(HERE, "host", "flux_driver.cpp"), "-o", exe, "-lm"],
                   check=True, capture_output=True)
    return exe


def run(exe, cmd, rows):
    text = "%s %d\n" % (cmd, len(rows)) + "\n".join(" ".join(float(v).hex() for v in r) for r in rows) + "\n"
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
    return np.array([[float.fromhex(v) for v in line.split()] for line in out.splitlines()])


def ln_mean(x, y):
    x, y = np.longdouble(x), np.longdouble(y)
    lo, hi = (x, y) if abs(x) < abs(y) else (y, x)
    d = (hi - lo) / lo
    return x if x == y else (hi - lo) / (np.log1p(d) if d < 1 else np.log(hi / lo))


def test_log_means(driver):
    rng = np.random.default_rng(3)
    x = 10.0 ** rng.uniform(-12, 3, 4000)
    ratio = np.concatenate([1.0 + 10.0 ** rng.uniform(-15, 0, 2000), 10.0 ** rng.uniform(0, 12, 2000)])
    y = np.where(rng.random(4000) < 0.5, x * ratio, x / ratio)
    sign = np.where(np.arange(4000) % 7 == 0, -1.0, 1.0)  # two negative values as well
    rows = np.stack([sign * x, sign * y], 1)
    got = run(driver, "means", rows)
    ref = np.array([ln_mean(a, b) for a, b in rows])
    # a rounded sum, difference, quotient, polynomial or logarithm (of a ratio
    # of 1.33 or more: its rounding counts up to 3.5 times) and product
    for k, r in ((0, ref), (1, 1 / ref), (2, ref), (3, 1 / ref)):
        err = np.abs(got[:, k] - r) / np.abs(r)
        print("mean %d: %.2f eps" % (k, float(err.max()) / EPS))
        assert err.max() < 8 * EPS


def test_log_mean_edges(driver):
    equal = [1e-9, 1.0, -1e-9, -3.0, -1e-300]
    got = run(driver, "means", [(v, v) for v in equal])
    assert np.all(np.abs(got[:, 2] - equal) <= EPS * np.abs(equal)), got
    assert np.all(np.abs(got[:4, 3] * equal[:4] - 1.0) <= 4 * EPS), got
    got = run(driver, "means", [(0.0, 0.0), (0.0, 2.0), (2.0, 0.0), (0.0, -2.0), (0.0, 1e-290)])
    assert np.all(got[:, 2] == 0.0), got
    got = run(driver, "means", [(1.0, -1.0), (-1e-9, 1.0), (1.0, -1e-9), (2.0, -1.0), (-1e-3, 0.7)])
    assert np.all(np.isnan(got[:, 2:])), got


def ec_energy(theta, R, TL, TR):
    theta, R, TL, TR = (np.longdouble(v) for v in (theta, R, TL, TR))
    bL, bR = 1 / TL, 1 / TR
    z = theta * (bR - bL) / 2
    sinhc = np.where(np.abs(z) < 1e-4, 1 + z * z / 6, np.sinh(z) / np.where(z == 0, 1, z))
    t = np.exp(-theta * (bL + bR) / 2) * sinhc / ln_mean(-np.expm1(-theta * bL), -np.expm1(-theta * bR))
    return R * (theta * t + 2.5 / ln_mean(bL, bR)) + 0.5 + 2 * R / (bL + bR)


@pytest.mark.parametrize("T", [100.0, 300.0, 1500.0, 6000.0, 2e4, 1e5, 1e6])
def test_ec_energy_mean(driver, T):
    rng = np.random.default_rng(4)
    rows = np.stack([rng.uniform(2200.0, 3400.0, 1000), np.full(1000, 297.0), T * np.exp(rng.uniform(-0.3, 0.3, 1000)),
                     T * np.exp(rng.uniform(-0.3, 0.3, 1000))], 1)
    got = run(driver, "ec", rows)[:, 0]
    ref = np.array([ec_energy(*r) for r in rows])
    err = float((np.abs(got - ref) / ref).max())
    print("T %g: %.2f eps" % (T, err / EPS))
    # two exponentials, their series, three means, three products and sums,
    # each within one unit of its last digit, and half a unit of beta = 1/T
    assert err < 10 * EPS


def test_two_point_fluxes_are_symmetric(driver):
    out = subprocess.run([driver], input="swap 2000\n", capture_output=True, text=True, check=True).stdout.split()
    print("pairs of 2000 whose flux depends on their order:", out)
    assert out == ["0"] * 10
