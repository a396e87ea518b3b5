"""Every shape of the column kernels over the column lengths, against the FP64
oracle: one to many columns per wavefront, the shapes that hand their two
transforms to two halves of a block, the ones that fall back where a length
does not allow them, with the inertial and the Stokes flow.  Three steps;
1e-10 as in the other parity tests (FP64 rounding, 1e-16, over the transforms
of a few steps), FP32 2e-5 and 2e-4 as there.
"""
from __future__ import annotations

import functools

import numpy as np
import pytest

from oracle import model_h as mh
from paper_0710_5912_amd import inputs

pytestmark = pytest.mark.gpu

le = pytest.importorskip("paper_0710_5912_amd.le")


def rel(a, b):
    den = np.max(np.abs(b))
    return float(np.max(np.abs(a - b)) / (den if den > 0 else 1.0))


def tol(precision, k):
    return 1e-10 if precision == "fp64" else 2e-5 if k == "phi" else 2e-4


@functools.lru_cache(maxsize=2)
def case(ny, rho):
    # sheared square grids up to 1024; above, narrow ones, which carry no shear
    nx = ny if ny <= 1024 else 16
    p = dict(nx=nx, ny=ny, lx=float(nx), ly=float(ny), gdot=4.0 / ny if nx == ny else 0.0, A=1.0,
             B=1.0, kappa=1.0, M=1.0, eta=1.0, rho=rho, dt=0.005)
    phi0 = inputs.noise_phi0(ny, nx, 71, amp=0.5)
    om0 = inputs.noise_omega0(ny, nx, 71) if rho > 0 else None
    op = mh.Params(**p)
    return p, phi0, om0, mh.run(op, mh.initial_state(op, phi0, om0), 3)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("variant", range(5))
@pytest.mark.parametrize("ny", [8, 16, 64, 128, 512, 1024, 2048, 4096])
def test_column_shapes(ny, variant, precision, monkeypatch):
    print(f"case ny={ny} variant {variant} {precision}", flush=True)
    monkeypatch.setenv("LE_TUNE_COL_CH", str(variant))
    monkeypatch.setenv("LE_TUNE_COL_FLOW", str(variant))
    # FP32 without the Stokes flow, whose psi carries phi's rounding times the
    # fourth power of the longest wave: no fixed bound over these lengths
    for rho in (1.0, 0.0) if precision == "fp64" else (1.0,):
        p, phi0, om0, st = case(ny, rho)
        with le.Context(p, phi0, om0, precision=precision) as c:
            c.step(3)
            g = c.get_state()
        for k in ("phi", "psi") + (("omega",) if rho > 0 else ()):
            assert rel(g[k], getattr(st, k)) <= tol(precision, k), (rho, k)
