"""The noise's logarithm and cosine (csrc/math64.h, compiled for the host)
against 64-bit-mantissa arithmetic: each within what its last rounding and the
terms before it leave."""

import os
import subprocess

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_11709_amd", "csrc")

PROGRAM = r"""
#include "math64.h"
#include <stdio.h>
int main() {
  double x;
  while (scanf("%la", &x) == 1) printf("%a %a\n", xrd::log_64(x), xrd::cos_rev64(x));
}
"""


def test_errors(tmp_path):
    src, exe = tmp_path / "n.cpp", tmp_path / "n"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC, str(src), "-o", str(exe)])
    rng = np.random.default_rng(6)
    one = 1.0 - 2.0 ** -np.arange(2.0, 54.0)
    x = np.concatenate([rng.random(60000), np.exp(-rng.uniform(0, 36, 20000)), one, 2.0 ** -np.arange(1.0, 55.0),
                        0.25 + (one - 1.0) / 2, 0.75 - (one - 1.0) / 4, rng.uniform(0.7, 0.7142, 20000)])
    out = subprocess.run([str(exe)], input="\n".join(float(v).hex() for v in x), capture_output=True, text=True,
                         check=True).stdout
    lg, cs = np.array([[float.fromhex(v) for v in line.split()] for line in out.splitlines()]).T
    L, u = np.longdouble, np.longdouble(2.0) ** -53
    want = np.log(x.astype(L))
    # the last rounding; the series' term, below a hundredth of the rest, at a few units
    assert np.max(np.abs((lg - want) / want)) <= 1.1 * u
    # the square's rounding moves the sine by 0.7 units at most, the small
    # terms' product and the last sum round once each, the coefficient of x^3 half
    n = np.rint(2 * x)
    r = 0.5 - np.abs(2 * x - n)  # exact
    pi = L(np.pi) + L(1.2246467991473532e-16)
    want = np.where(n == 1.0, -1, 1) * np.sin(pi * r.astype(L))
    on = r != 0
    assert not cs[~on].any()
    assert np.max(np.abs((cs[on] - want[on]) / want[on])) <= 2 * u
