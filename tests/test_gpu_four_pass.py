"""The four-pass row kernels (inverse row transforms inside the stencil
kernels) against the FP64 oracle.

They run wherever no kernel variant is fixed, in three shapes: two rows per
block with 4 values per thread (short rows), two and four rows with 8 or 16.
The grids sit on both sides of every line between the shapes, with halo rows
that wrap (ny = 8), row lengths from one wavefront's part to several segments
per thread, and every kind of diagonal: r = 1 with both signs of the strain
offset, even r, and r = 0 (nx < ny, unsheared).  Two rounds of 1e-10 as in the
other parity tests (FP64 rounding, 1e-16, over the transforms of a few dozen
steps); FP32 2e-5 and 2e-4 as there.
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import model_h as mh
from paper_0710_5912_amd import inputs

pytestmark = pytest.mark.gpu

le = pytest.importorskip("paper_0710_5912_amd.le")


def rel(a, b):
    den = np.max(np.abs(b))
    return float(np.max(np.abs(a - b)) / (den if den > 0 else 1.0))


def case(nx, ny, gdot, rho, **kw):
    p = dict(nx=nx, ny=ny, lx=float(nx), ly=float(ny), gdot=gdot, A=1.0, B=1.0, kappa=1.0, M=1.0,
             eta=1.0, rho=rho, dt=0.005)
    phi0 = inputs.noise_phi0(ny, nx, 51, amp=0.5)
    om0 = inputs.noise_omega0(ny, nx, 51) if rho > 0 else None
    op = mh.Params(**p, **kw)
    return p, phi0, om0, op


GRIDS = [(8, 8, 3.0, 60), (16, 8, -2.0, 60), (8, 64, 0.0, 4), (64, 64, -0.4, 20),
         (256, 16, 0.5, 40), (512, 256, 0.2, 4), (512, 512, -0.3, 3), (512, 1024, 0.0, 2),
         (512, 2048, 0.0, 1), (1024, 128, 0.1, 3), (1024, 1024, -0.1, 2), (2048, 256, 0.1, 2),
         (2048, 512, -0.1, 2), (2048, 1024, 0.1, 1)]


@pytest.mark.parametrize("rho", [1.0, 0.0])
@pytest.mark.parametrize("nx,ny,gdot,steps", GRIDS)
def test_four_pass_fp64(nx, ny, gdot, steps, rho):
    p, phi0, om0, op = case(nx, ny, gdot, rho)
    print(f"case {nx}x{ny} gdot={gdot} rho={rho} steps={steps}", flush=True)
    st = mh.run(op, mh.initial_state(op, phi0, om0), steps)
    with le.Context(p, phi0, om0) as c:
        c.step(steps)
        g = c.get_state()
    assert g["wraps"] == st.wraps
    for k in ("phi", "psi") + (("omega",) if rho > 0 else ()):
        assert rel(g[k], getattr(st, k)) <= 1e-10, k


@pytest.mark.parametrize("nx,ny,gdot", [(64, 32, 0.4), (512, 512, -0.3), (1024, 256, 0.1),
                                        (1024, 1024, 0.1), (2048, 1024, -0.1), (2048, 2048, 0.1)])
def test_four_pass_fp32(nx, ny, gdot):
    p, phi0, om0, op = case(nx, ny, gdot, 1.0)
    print(f"case {nx}x{ny} gdot={gdot} fp32", flush=True)
    st = mh.run(op, mh.initial_state(op, phi0, om0), 3)
    with le.Context(p, phi0, om0, precision="fp32") as c:
        c.step(3)
        g = c.get_state()
    assert rel(g["phi"], st.phi) <= 2e-5
    assert rel(g["psi"], st.psi) <= 2e-4


@pytest.mark.parametrize("nx,ny", [(128, 32), (1024, 128)])
def test_four_pass_f_half(nx, ny):
    """f of the advected phi in a narrow and a wide shape."""
    p, phi0, om0, op = case(nx, ny, 0.3, 1.0, f_half=True)
    st = mh.run(op, mh.initial_state(op, phi0, om0), 3)
    with le.Context(p, phi0, om0) as c:
        c.set_scheme(f_half=True)
        c.step(3)
        g = c.get_state()
    for k in ("phi", "omega", "psi"):
        assert rel(g[k], getattr(st, k)) <= 1e-10, k


def test_four_pass_batch_equals_single_runs(monkeypatch):
    """Every run of a batch equals its run alone bit for bit (the columns'
    shapes fixed, the row kernels' shape a function of the grid)."""
    monkeypatch.setenv("LE_TUNE_COL_CH", "0")
    monkeypatch.setenv("LE_TUNE_COL_FLOW", "0")
    runs = [(case(n, n, g, rho)[0], inputs.noise_phi0(n, n, 60 + i, amp=0.4))
            for i, (n, g, rho) in enumerate([(64, 0.4, 1.0), (512, -0.3, 1.0), (64, -0.2, 1.0),
                                             (512, 0.1, 1.0), (128, 0.3, 0.0)])]
    b = le.Batch([r[0] for r in runs], [r[1] for r in runs])
    b.step(20)
    for i, (p, phi0) in enumerate(runs):
        with le.Context(p, phi0) as c:
            c.step(20)
            ref = c.get_state()
        got = b.get_state(i)
        for k in ("phi", "omega", "psi"):
            assert np.array_equal(got[k], ref[k]), (i, k)
    b.close()
