"""The table functions' errors (csrc/math64.h, compiled for the host) against
64-bit-mantissa arithmetic: e^x to the same few units at every x, e^{-B s2} as
good as its one rounded factor, sin and cos to one and a half units."""

import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_11709_amd", "csrc")
U = np.longdouble(2.0) ** -53

PROGRAM = r"""
#include "math64.h"
#include <math.h>
#include <stdio.h>
using namespace xrd;
static Rev64 rev[kRev];
static double e2[kExp2];
int main() {
  for (int k = 0; k <= kRev / 2; ++k) {
    const long double a = 2.0L * acosl(-1.0L) * k / kRev;
    rev[k] = Rev64{(double)(k == kRev / 4 ? 0.0L : cosl(a)), (double)(k == kRev / 2 ? 0.0L : sinl(a))};
    if (k > 0 && k < kRev / 2) rev[kRev - k] = Rev64{rev[k].c, -rev[k].s};
  }
  for (int k = 0; k < kExp2; ++k) e2[k] = (double)exp2l((long double)k / kExp2);
  double x, y;
  while (scanf("%la %la", &x, &y) == 2) {
    double s, c;
    sincos_tab64(kRev * x, rev, &s, &c);
    printf("%a %a %a %a\n", exp_tab64(x, e2), exp2_tab64(x, e2, tab_exponent64(-y)), s, c);
  }
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("math64")
    (d / "m.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC, str(d / "m.cpp"), "-o",
                           str(d / "m")])

    def go(x, y):
        text = "\n".join(f"{float(a).hex()} {float(b).hex()}" for a, b in zip(x, y))
        out = subprocess.run([str(d / "m")], input=text, capture_output=True, text=True, check=True).stdout
        return np.array([[float.fromhex(v) for v in line.split()] for line in out.splitlines()]).T
    return go


@pytest.mark.parametrize("span", [1.0, 20.0, 300.0])
def test_exponentials(run, span):
    rng = np.random.default_rng(int(span))
    x = rng.uniform(-span, span, 20000)
    s2 = rng.uniform(0.0, 2.0, 20000)
    e, w, _, _ = run(x, s2)
    X = x.astype(np.longdouble)
    want = np.exp(X)
    # the table's power and the last sum, a unit each, and the polynomial's 0.4
    assert np.max(np.abs((e - want) / want)) <= 2.4 * U
    arg = -X * s2.astype(np.longdouble)
    want = np.exp(arg)
    assert np.all(np.abs((w - want) / want) <= (2.4 + np.abs(arg)) * U)


def test_circular_functions(run):
    rng = np.random.default_rng(5)
    t = np.concatenate([rng.uniform(-0.5, 0.5, 40000), (np.arange(512) + 0.5) / 512, np.arange(512) / 512])
    _, _, s, c = run(t, np.ones(len(t)))
    pi = np.longdouble(np.pi) + np.longdouble(1.2246467991473532e-16)
    r = t - np.rint(t)
    # the table's rounding and two sums', half a unit each; the small angle's own
    assert np.max(np.abs(s - np.sin(2 * pi * r.astype(np.longdouble)))) <= 1.52 * U
    assert np.max(np.abs(c - np.cos(2 * pi * r.astype(np.longdouble)))) <= 1.52 * U


def test_circular_functions_near_their_zeros(run):
    """Relative there: the table's rotations by quarters are exact."""
    d = 2.0 ** -np.arange(11.0, 60.0)
    pi = np.longdouble(np.pi) + np.longdouble(1.2246467991473532e-16)
    for at in (0.0, 0.5, -1.0, 7.5):
        t = at + d
        left = t - at  # what the sum kept of d
        s = run(t, np.ones(len(t)))[2]
        want = np.sin(2 * pi * left.astype(np.longdouble)) * (-1 if at % 1 else 1)
        on = left != 0
        assert np.max(np.abs((s[on] - want[on]) / want[on])) <= 4 * U
