"""Advection in batches of eight rows (single precision, rows of 4096) against
batches of four: the same stencil and transforms per row, so the same bits, for
one batch and several per block, strips longer than the grid, and halo rows
that wrap onto the batch itself (ny = 8)."""
from __future__ import annotations

import numpy as np
import pytest

from paper_0710_5912_amd import inputs

pytestmark = pytest.mark.gpu

le = pytest.importorskip("paper_0710_5912_amd.le")


def run(ny, rho, variant, monkeypatch):
    print(f"case 4096x{ny} rho={rho} advect {variant}", flush=True)
    for k in ("COL_CH", "COL_FLOW", "ROW", "ROW_FWD"):
        monkeypatch.setenv("LE_TUNE_" + k, "0")
    monkeypatch.setenv("LE_TUNE_MU", "4")
    monkeypatch.setenv("LE_TUNE_ADV", str(variant))
    p = dict(nx=4096, ny=ny, lx=4096.0, ly=float(ny), gdot=0.1, A=1.0, B=1.0, kappa=1.0, M=1.0,
             eta=1.0, rho=rho, dt=0.005)
    phi0 = inputs.noise_phi0(ny, 4096, 81, amp=0.5)
    om0 = inputs.noise_omega0(ny, 4096, 81) if rho > 0 else None
    with le.Context(p, phi0, om0, precision="fp32") as c:
        c.step(2)
        return c.get_state()


@pytest.mark.parametrize("rho", [1.0, 0.0])
@pytest.mark.parametrize("ny", [8, 16, 64, 4096])
def test_eight_rows_equal_four(ny, rho, monkeypatch):
    ref = run(ny, rho, 132, monkeypatch)
    for variant in (136, 144):
        got = run(ny, rho, variant, monkeypatch)
        for k in ("phi", "omega", "psi"):
            assert np.array_equal(got[k], ref[k]), (variant, k)
