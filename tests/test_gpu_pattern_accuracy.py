"""The plain path's pattern of given reflections against 64-bit-mantissa
arithmetic, relative to each point and in the 2-norm, over the grids that the
ratio form takes (and one beside them), and its answer to intensities that are
not finite."""

import numpy as np
import pytest
import torch

from paper_2602_11709_amd import synth
from paper_2602_11709_amd.api import Grid, XrdBatch

pytestmark = pytest.mark.gpu

U = 2.0 ** -53
# A point: the offset, its square and the exponent's factor each round by U, of
# an exponent e <= window^2 / 2 <= 72 (four roundings: 288 U); the line's value
# and up to four ratios of it at 4 U a step, the factor at the end and the sum.
POINT = (288 + 4 * 4 + 6) * U
# The norm's weight lies where e <= 2.
NORM = (4 * 2 + 4 * 4 + 6) * U


def _reflections(friedel):
    xb = XrdBatch(synth.rocksalt(), precision="fp64", friedel=friedel, grid_capacity=8192)
    refl = xb.enumerate()
    return xb, refl, xb.structure_factors(refl)[2], int(xb.read_counts(refl)[0][-1])


@pytest.mark.parametrize("dt_sigmas", [0.05, 0.2, 0.35, 0.5, 0.6])
@pytest.mark.parametrize("sigma", [0.5, 0.1, 0.02, 0.001])
@pytest.mark.parametrize("window", [4.0, 8.0, 12.0])
def test_points_and_norm(sigma, dt_sigmas, window):
    xb, refl, I, n = _reflections(True)
    tt, v = refl.two_theta[:n].cpu().numpy(), I[:n].cpu().numpy()
    peak = float(tt[np.argmax(v)])
    dt = sigma * dt_sigmas
    grid = Grid(peak - 700.3 * dt, dt, 1501, sigma, window)
    y = xb.pattern_forward(refl, I, grid).cpu().numpy()[0]
    x = grid.t0 + np.arange(grid.n_points) * dt
    d = x[:, None] - tt[None, :]
    inside = np.abs(d) <= window * sigma
    L = np.longdouble
    s = L(sigma)
    K = np.where(inside, np.exp(-(x[:, None].astype(L) - tt[None, :].astype(L)) ** 2 / (2 * s * s)), L(0))
    want = (K * (v.astype(L) / (s * np.sqrt(2 * L(np.pi) + 2 * L(1.2246467991473532e-16))))[None, :]).sum(1)
    assert not y[want == 0].any()
    on = want > 0
    point = float(np.max(np.abs(y[on] - want[on]) / want[on]))
    norm = float(np.sqrt(((y - want) ** 2).sum() / (want ** 2).sum()))
    print(f"sigma {sigma} dt/sigma {dt_sigmas} window {window}: point {point:.2e} norm {norm:.2e}", flush=True)
    assert point <= POINT and norm <= NORM


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_intensities_that_are_not_finite(bad):
    """Only the points of their own windows take them up."""
    xb, refl, I, n = _reflections(False)
    tt = refl.two_theta[:n].cpu().numpy()
    grid = Grid(20.0, 0.01, 6001, 0.05, 8.0)
    y0 = xb.pattern_forward(refl, I, grid).cpu().numpy()[0]
    j = int(np.argmax(I[:n].cpu().numpy()))
    I[j] = bad
    y = xb.pattern_forward(refl, I, grid).cpu().numpy()[0]
    x = grid.t0 + np.arange(grid.n_points) * grid.dt
    inside = np.abs(x - tt[j]) <= grid.window_sigmas * grid.sigma
    assert inside.any() and np.array_equal(y[~inside], y0[~inside])
    assert np.array_equal(y[inside], np.full(inside.sum(), bad), equal_nan=True)
