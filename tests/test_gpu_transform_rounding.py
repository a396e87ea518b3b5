"""Rounding of the FP64 transforms: a step so short that it changes nothing
(dt = 1e-30) returns phi after one forward and one inverse transform of the rows
and of the columns, so what differs is their rounding.

Each of the L = log2(points) radix-2 levels of a transform (one more joins or
splits the real row) rounds its sums and carries its twiddle's error, table
rounding (0.4 u RMS, u = 2^-53) doubled by at most one squaring, which enters
half of the data: together below u RMS a level, independent between levels.  So
the RMS difference is at most u sqrt(levels).  (Twiddles squared three times
carry 4 u into one level of a 16-point pass and exceed it.)
"""
from __future__ import annotations

import numpy as np
import pytest

from paper_0710_5912_amd import inputs

pytestmark = pytest.mark.gpu

le = pytest.importorskip("paper_0710_5912_amd.le")


@pytest.mark.parametrize("nx,ny,col", [(64, 64, None), (512, 512, None), (512, 64, 1), (64, 512, 0),
                                       (64, 512, 3), (1024, 1024, None), (2048, 256, None),
                                       (2048, 1024, 1), (2048, 2048, 0), (4096, 64, None),
                                       (16, 2048, 0), (16, 4096, 0), (16, 4096, 1)])
def test_round_trip(nx, ny, col, monkeypatch):
    print(f"case {nx}x{ny} column shape {col}", flush=True)
    if col is not None:
        monkeypatch.setenv("LE_TUNE_COL_CH", str(col))
        monkeypatch.setenv("LE_TUNE_COL_FLOW", str(col))
    p = dict(nx=nx, ny=ny, lx=float(nx), ly=float(ny), gdot=0.0, A=1.0, B=1.0, kappa=1.0, M=1.0,
             eta=1.0, rho=1.0, dt=1e-30)
    phi0 = inputs.noise_phi0(ny, nx, 91, amp=0.5)
    with le.Context(p, phi0) as c:
        c.step(1)
        phi = c.get_state()["phi"]
    levels = 2 * np.log2(nx * ny)
    d = np.sqrt(np.mean((phi - phi0) ** 2) / np.mean(phi0 ** 2))
    print(f"  {d * 2.0 ** 53 / np.sqrt(levels):.2f} u per level", flush=True)
    assert d <= 2.0 ** -53 * np.sqrt(levels)
