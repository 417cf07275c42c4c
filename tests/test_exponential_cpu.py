"""The exponential of the vocabulary reduction (csrc/k_exp.h), built for the CPU: its formula against 64 bits.  The hardware's
2^t stands in as the correctly rounded one."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_18489_amd", "csrc")
MAIN = r"""
#include <math.h>
#include <stdio.h>
#define __device__
#define __forceinline__ inline
static float two_to(float t) { return (float)exp2((double)t); }
#define __builtin_amdgcn_exp2f two_to
#include "k_exp.h"
int main() {
  float d;
  while (fread(&d, 4, 1, stdin) == 1) { const float e = ec::exp_of_negative(d); fwrite(&e, 4, 1, stdout); }
}
"""


@pytest.fixture(scope="module")
def exp_of_negative(tmp_path_factory):
    at = tmp_path_factory.mktemp("exp")
    (at / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-O1", "-ffp-contract=off", "-I", CSRC, str(at / "main.cpp"), "-o", str(at / "exp")])
    return lambda d: np.frombuffer(subprocess.run([str(at / "exp")], input=d.astype(np.float32).tobytes(),
                                                  stdout=subprocess.PIPE, check=True).stdout, dtype=np.float32)


@pytest.mark.parametrize("lo,hi", [(-1, 0), (-5, -1), (-10, -5), (-20, -10), (-50, -20), (-87, -50)])
def test_formula_is_as_exact_as_float32_allows(exp_of_negative, lo, hi):
    """Two roundings, of 2^t and of the last sum, are 2^-24 each; the corrected remainder (|r| below 8e-6) adds r^2 / 2 < 4e-11
    and its own rounding.  Neither rounding has a side: the mean over 20000 arguments stays under five standard deviations
    of it, 5 * 2^-24 * sqrt(2 / 3 / 20000) < 1.8e-9, and the 2.2e-9 by which results above 1/e, whose 2^t the last
    sum often returns unchanged, are off to one side.  (A remainder that forgets the low part of ln 2 has 9e-9 from -5 to
    -1, 1.9e-7 from -87 to -50.)"""
    d = np.random.default_rng(7).uniform(lo, hi, 20000).astype(np.float32)
    err = exp_of_negative(d).astype(np.float64) / np.exp(d.astype(np.float64)) - 1.0
    print(err.mean(), np.abs(err).max())
    assert np.abs(err).max() < 2.0 ** -23 * 1.01
    assert abs(err.mean()) < 4e-9


def test_ends_of_the_range(exp_of_negative):
    got = exp_of_negative(np.array([0.0, -2.0 ** -30, -200.0]))
    assert got[0] == 1.0 and got[1] == 1.0 and got[2] == 0.0
