"""The step's joined row kernels where a caller compares runs bit for bit, and
their timing.  No kernel variant is fixed here, so the joined kernels run on every
grid that has them (contexts of one shape share their other kernels in a process):
64 x 64 and 64 x 32 have narrow shapes, 1024 x 128 a wide one, 2048 x 128 only
stages 3 and 4 joined.
"""
from __future__ import annotations

import numpy as np
import pytest

from paper_0710_5912_amd import inputs

pytestmark = pytest.mark.gpu

le = pytest.importorskip("paper_0710_5912_amd.le")

FLOW, MU = ("row_inv_flow", "advect"), ("row_inv_phi", "mu_source")
GRIDS = [(64, 64, "fp64", 1.0), (64, 32, "fp64", 0.0), (64, 64, "fp32", 1.0),
         (1024, 128, "fp64", 1.0), (1024, 128, "fp32", 0.0), (2048, 128, "fp64", 1.0)]


def params(nx, ny, rho, gdot):
    return dict(nx=nx, ny=ny, lx=float(nx), ly=float(ny), gdot=gdot, A=1.0, B=1.0, kappa=1.0,
                M=1.0, eta=1.0, rho=rho, dt=0.005)


def make(nx, ny, precision, rho, gdot=0.5, amp=0.5):
    print(f"case {nx}x{ny} {precision} rho={rho}", flush=True)
    return le.Context(params(nx, ny, rho, gdot), inputs.noise_phi0(ny, nx, 61, amp=amp),
                      precision=precision)


def same(a, b):
    ga, gb = a.get_state(), b.get_state()
    assert ga["step"] == gb["step"] and ga["wraps"] == gb["wraps"]
    for k in ("phi", "omega", "psi"):
        assert np.array_equal(ga[k], gb[k]), k


@pytest.mark.parametrize("nx,ny,precision,expect", [
    (8, 8, "fp64", [FLOW, MU]), (1024, 128, "fp64", [FLOW, MU]), (2048, 128, "fp64", [MU]),
    (2048, 512, "fp64", [FLOW, MU]), (2048, 2048, "fp64", []), (2048, 2048, "fp32", [MU]),
    (4096, 16, "fp64", [])])
def test_joined_stages(nx, ny, precision, expect, monkeypatch):
    with make(nx, ny, precision, 1.0, gdot=0.0) as c:
        assert c.joined() == expect
        c.set_scheme(upwind3=True)
        assert c.joined() == [p for p in expect if p != FLOW]
    monkeypatch.setenv("LE_TUNE_ROW", "0")
    with make(nx, ny, precision, 1.0, gdot=0.0) as c:
        assert c.joined() == []


@pytest.mark.parametrize("nx,ny,precision,rho", GRIDS)
def test_timing_leaves_the_steps(nx, ny, precision, rho):
    """Timed steps, and steps after every stage timed in any order, equal untimed ones."""
    with make(nx, ny, precision, rho) as a, make(nx, ny, precision, rho) as b:
        a.profile(True)
        a.step(20)
        times = a.stage_times()
        a.profile(False)
        b.step(20)
        same(a, b)
        assert all(n == 20 and ms > 0.0 for ms, n in times.values()), times
        for pair in a.joined():
            assert times[pair[0]][0] == times[pair[1]][0]
        for s in le.STAGES[::-1] + le.STAGES:
            assert a.time_stage(s, 2) > 0.0
        same(a, b)
        a.step(7)
        b.step(7)
        same(a, b)


@pytest.mark.parametrize("nx,ny,precision,rho", GRIDS)
def test_graph_pieces_equal_eager_launches(nx, ny, precision, rho, monkeypatch):
    monkeypatch.setenv("LE_GRAPHS", "0")
    eager = make(nx, ny, precision, rho)
    monkeypatch.setenv("LE_GRAPHS", "1")
    graph = make(nx, ny, precision, rho)
    with eager, graph:
        for n in (37, 128, 5, 77, 1, 40):
            eager.step(n)
            graph.step(n)
            same(eager, graph)
            assert eager.observables()[0]["Ls"] == graph.observables()[0]["Ls"]


@pytest.mark.parametrize("nx,ny,precision,rho", GRIDS)
def test_checkpoint_resume_is_bitwise(nx, ny, precision, rho):
    with make(nx, ny, precision, rho) as a, make(nx, ny, precision, rho) as b:
        a.step(25)
        blob = a.checkpoint()
        a.step(30)
        b.step(3)
        b.restore(blob)
        b.step(30)
        same(a, b)


@pytest.mark.parametrize("nx,ny,precision,rho", GRIDS)
def test_recovery_stops_at_the_last_finite_step(nx, ny, precision, rho):
    """An explicit step far beyond its stable size: the call stops at the last finite
    step, with the state of a run of that many steps."""
    p = dict(params(nx, ny, rho, 0.01), kappa=0.01, dt=1.0)
    phi0 = inputs.noise_phi0(ny, nx, 62, amp=0.05)
    with le.Context(p, phi0, precision=precision) as a, \
            le.Context(p, phi0, precision=precision) as b:
        print(f"case {nx}x{ny} {precision} rho={rho}", flush=True)
        with pytest.raises(le.LeError) as ei:
            a.step(500)
        assert ei.value.code == le.LE_ENONFINITE
        g = a.get_state()
        assert 0 < g["step"] < 500 and np.all(np.isfinite(g["phi"]))
        b.step(g["step"])
        gb = b.get_state()
        for k in ("phi", "omega", "psi"):
            assert np.array_equal(g[k], gb[k], equal_nan=True), k
        with pytest.raises(le.LeError) as ei:
            b.step(1)
        assert ei.value.code == le.LE_ENONFINITE


def test_corrected_steps_and_audits_are_bitwise(monkeypatch):
    """Corrected graph replays equal eager launches; a run whose audits pass equals
    the unaudited one, a run whose audit fails its plain continuation."""
    def corrected():
        c = make(64, 64, "fp64", 1.0, gdot=0.1)
        c.corrector_load(inputs.cnn_init_params(3), [1.0, 10.0, 0.05, 0.01])
        return c

    monkeypatch.setenv("LE_GRAPHS", "0")
    eager = corrected()
    monkeypatch.setenv("LE_GRAPHS", "1")
    with eager, corrected() as graph, corrected() as audited, corrected() as fails:
        assert eager.joined() == [FLOW, MU]
        audited.corrector_audit(10, 4, 1e9)
        for n in (33, 64, 7):
            for c in (eager, graph, audited):
                c.step_corrected(n)
            same(eager, graph)
            same(eager, audited)
        assert not audited.corrector_status()[0] and audited.corrector_status()[1] > 0
        fails.corrector_audit(6, 3, 0.0)
        fails.step_corrected(20)
        assert fails.corrector_status()[0]
        with corrected() as plain:
            plain.step_corrected(6)
            plain.step(14)
            same(fails, plain)


@pytest.mark.parametrize("nx,ny,gdot", [(512, 512, -0.3), (1024, 256, 0.1), (1024, 1024, 0.1),
                                        (2048, 1024, -0.1), (2048, 2048, 0.1)])
def test_fp32_stokes_in_the_wide_shapes(nx, ny, gdot, monkeypatch):
    """Single precision without inertia: phi within the FP32 bound of the other parity
    tests.  psi = g / lambda^2 is the rounding of g in its longest wave, which no fixed
    bound holds: against the oracle it is at most eight times what the stages' own
    kernels give (forms that round differently scatter by factors from 0.3 to 2)."""
    from oracle import model_h as mh

    p, phi0 = params(nx, ny, 0.0, gdot), inputs.noise_phi0(ny, nx, 51, amp=0.5)
    op = mh.Params(**p)
    st = mh.run(op, mh.initial_state(op, phi0, None), 3)
    err = []
    for joined in (True, False):
        if not joined:
            monkeypatch.setenv("LE_TUNE_ROW", "0")
        print(f"case {nx}x{ny} joined={joined}", flush=True)
        with le.Context(p, phi0, precision="fp32") as c:
            assert c.joined() == ([FLOW, MU] if joined else [])
            c.step(3)
            g = c.get_state()
        assert np.max(np.abs(g["phi"] - st.phi)) <= 2e-5 * np.max(np.abs(st.phi))
        err.append(np.max(np.abs(g["psi"] - st.psi)) / np.max(np.abs(st.psi)))
    print(f"  psi {err[0]:.2e}, apart {err[1]:.2e}", flush=True)
    assert err[0] <= 8.0 * err[1]
