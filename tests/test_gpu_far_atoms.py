"""Atoms given many cells away (coordinates up to 2^44) scatter like the same
atoms in the first cell: structure factors and gradients, both methods.  The
coordinates are multiples of 1/64, so every phase is exact before its
reduction; what remains is the sums' rounding."""

import dataclasses

import numpy as np
import pytest
import torch

from paper_2602_11709_amd import synth
from paper_2602_11709_amd.api import Grid, XrdBatch

pytestmark = pytest.mark.gpu

GRID = Grid(10.0, 0.05, 1600, 0.1)


def _run(b, precision, method):
    xb = XrdBatch(b, precision=precision, sf_method=method, grid_capacity=GRID.n_points, keep_sf_derivs=True)
    refl = xb.enumerate()
    A, B, I = xb.structure_factors(refl)
    n = int(xb.read_counts(refl)[0][-1])
    xb.pattern_forward(refl, I, GRID)
    dy = torch.cos(0.01 * torch.arange(GRID.n_points, dtype=torch.float64, device="cuda")).repeat(b.n_crystals, 1)
    grads = xb.pattern_backward(refl, GRID, dy)
    return [t.double().cpu().numpy() for t in (A[:n], B[:n], *grads)]


@pytest.mark.parametrize("cells", [2.0 ** 19, -(2.0 ** 21), 2.0 ** 44])
@pytest.mark.parametrize("method", ["direct", "recurrence"])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_far_atoms(precision, method, cells):
    b = synth.random_triclinic(17, 4, len_hi=9.0, atoms_lo=5, atoms_hi=70)
    frac = np.round(b.frac * 64.0) / 64.0
    near = dataclasses.replace(b, frac=frac)
    far = dataclasses.replace(b, frac=frac + cells * np.array([1.0, -1.0, 2.0 ** -1]))
    # double: a thousand roundings of 2^-53; mixed: its single-precision phases
    # (2^-24 of a revolution) and sums of up to 70 terms
    tol = 1e-12 if precision == "fp64" else 5e-5
    for name, p, q in zip(("A", "B", "dfrac", "dbfac", "dlat"), _run(near, precision, method),
                          _run(far, precision, method)):
        err = np.max(np.abs(p - q)) / np.max(np.abs(p))
        print(precision, method, cells, name, f"{err:.2e}", flush=True)
        assert err <= tol, name
