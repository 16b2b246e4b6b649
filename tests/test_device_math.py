"""The device's logarithms and exponential (csrc/device/math.hip), the functions
themselves compiled for the host (the hardware's reciprocal estimate as 1/x),
against 80-bit ones.  No GPU.

Tolerances: ln 2 ulp, as derived in test_ln, and for lg one more for the product
with 1/ln 10; exp_neg 2 ulp (polynomial and reduction 1.5)."""
import pathlib
import subprocess

import numpy as np
import pytest

import hostemu_build as hb

MATH = pathlib.Path(__file__).resolve().parents[1] / "paper_2508_16105_amd" / "csrc" / "device" / "math.hip"
DRIVER = r"""
#include "shim.h"
#include <stdio.h>
namespace chem_config { constexpr bool kExpSaturatingConvert = SAT; }
#include MATH
emu_dim3 threadIdx, blockIdx, blockDim, gridDim;
double* emu_lds;
int main(int argc, char** argv)
{
    double x, r[8];
    while (fread(&x, 8, 1, stdin) == 1) {
        const long double l = x, el = expl(l), ll = logl(l), lt = log10l(l);
        r[0] = chem_math::ln(x); r[1] = chem_math::ln<true>(x); r[2] = chem_math::lg(x); r[3] = chem_math::exp_neg(x);
        // errors of the four in units in the last place of the double nearest the reference
        const long double ref[4] = {ll, ll, lt, el};
        for (int k = 0; k < 4; ++k) {
            const double d = (double)ref[k], u = nextafter(fabs(d), INFINITY) - fabs(d);
            r[4 + k] = d == 0.0 ? (r[k] == 0.0 ? 0.0 : INFINITY) : (double)(fabsl((long double)r[k] - ref[k]) / u);
        }
        fwrite(r, 8, 8, stdout);
    }
}
"""


@pytest.fixture(scope="module", params=[False, True], ids=["clamped", "saturating"])
def functions(request, tmp_path_factory):
    if not pathlib.Path(hb.CLANG).exists():
        pytest.skip("host clang++ not available")
    wd = tmp_path_factory.mktemp("math")
    text = MATH.read_text().replace("__builtin_amdgcn_rcp(", "1.0 / (")
    text = text.replace('asm("v_cvt_i32_f64 %0, %1" : "=v"(n) : "v"(nd));', "n = emu_cvt_i32_sat(nd);")
    (wd / "math.inc").write_text(text)
    (wd / "driver.cpp").write_text(DRIVER)
    exe = wd / "driver"
    subprocess.run([hb.CLANG, "-x", "c++", "-std=c++17", "-O1", "-ffp-contract=off", "-mfma",
                    f"-DSAT={str(request.param).lower()}", f'-DMATH="{wd / "math.inc"}"', f"-I{hb.EMU}",
                    str(wd / "driver.cpp"), "-o", str(exe), "-lm"], check=True, capture_output=True, text=True)

    def run(x):
        r = subprocess.run([str(exe)], input=np.asarray(x, dtype=np.float64).tobytes(), check=True, capture_output=True)
        return np.frombuffer(r.stdout).reshape(-1, 8)
    return run


@pytest.mark.parametrize("lo,hi", [(0.5, 2.0), (200.0, 6000.0), (1e-300, 1e300)])
def test_logarithms_of_normal_numbers(functions, lo, hi):
    x = np.exp(np.random.default_rng(1).uniform(np.log(lo), np.log(hi), 20000))
    if lo < 1.0 < hi:
        x = np.concatenate([x, 1.0 + np.random.default_rng(2).uniform(-1e-6, 1e-6, 2000),
                            [1.0, np.nextafter(1.0, 0.0), np.nextafter(1.0, 2.0)]])
    r = functions(x)
    assert r[:, 4].max() <= 2.0 and r[:, 5].max() <= 2.0 and r[:, 6].max() <= 3.0
    assert np.array_equal(r[:, 0], r[:, 1])


def test_logarithms_of_subnormal_numbers(functions):
    x = np.ldexp(np.random.default_rng(3).uniform(0.5, 1.0, 2000), np.random.default_rng(4).integers(-1073, -1021, 2000))
    x = np.concatenate([x, [5e-324, 2.2250738585072014e-308]])
    r = functions(x)
    assert r[:, 5].max() <= 2.0 and r[:, 6].max() <= 3.0


def test_exponential(functions):
    x = np.concatenate([-np.random.default_rng(5).uniform(0.0, 700.0, 20000),
                        -np.exp(np.random.default_rng(6).uniform(-40.0, 6.0, 5000)), [0.0, -0.0]])
    assert functions(x)[:, 7].max() <= 2.0
    assert np.array_equal(functions([-800.0, -1e4, -1e300, -np.inf])[:, 3], np.zeros(4))


def test_what_has_no_logarithm_is_not_a_number(functions):
    r = functions([0.0, -0.0, -1.0, -1e300, np.inf, -np.inf, np.nan])
    assert np.isnan(r[:, :3]).all()
    assert np.isnan(functions([np.nan, np.inf])[:, 3]).all()
