"""The planner's FP32 schedules (lifts formed from terms in the stages, split up
to 2^19 points, the inverse iteration with its own lift launch), executed by the
numpy interpreter in FP64 against the oracle at the bar of test_plan_lifts.py."""
import json
import math
import subprocess

import pytest

import plan_interp
from oracle.hos import Grid, HOSModel
from paper_2608_25203_amd.inputs import random_band_fields
from plan_interp import Interp
from test_host import rel
from test_plan_lifts import run_fused

TWO_PI = 2 * math.pi


@pytest.fixture(autouse=True)
def fp32_plans(monkeypatch):
    def load(nx, ny, M, eps=1.0, taper=True, filt=True, dt=1.0):
        out = subprocess.run([plan_interp.build_checker(), str(nx), str(ny), str(M), repr(float(eps)), str(int(taper)),
                              str(int(filt)), repr(float(dt)), "32"], capture_output=True, text=True, check=True)
        return json.loads(out.stdout)

    monkeypatch.setattr(plan_interp, "load_plan", load)


# 640 x 512 lies between the FP64 and FP32 merge lines, 1024 x 640 above both
@pytest.mark.parametrize("ab2", [False, True])
@pytest.mark.parametrize("nx,ny,M", [(32, 32, 1), (32, 32, 2), (32, 48, 3), (48, 32, 5), (64, 1, 3), (32, 32, 8),
                                     (640, 512, 2), (1024, 640, 2)])
def test_fp32_steps_match_oracle(nx, ny, M, ab2):
    Lx, Ly = TWO_PI * nx / 32, (TWO_PI * ny / 32 if ny > 1 else 1.0)
    eta, psi = random_band_fields(nx, ny, 60 + M, 5, amplitude=0.02)
    I = Interp(nx, ny, Lx, Ly, 0.8, 9.81, M)
    m = HOSModel(Grid(nx, ny, Lx, Ly, 0.8), M)
    ref = (m.step_ifab2 if ab2 else m.step)(eta, psi, 0.004, 2)
    for a, b in zip(run_fused(I, eta, psi, 0.004, 2, ab2), ref):
        assert rel(a, b) < 1e-13


@pytest.mark.parametrize("M", [1, 2, 3, 4])
def test_fp32_inverse_iteration_is_the_fp64_one(monkeypatch, M):
    """psi + G0^-1 (v - G psi), lifted by a launch of its own, against the FP64
    plan's G0^-1 (v - (G - G0) psi): the same iterates to rounding."""
    nx = ny = 32
    eta, v = random_band_fields(nx, ny, 70 + M, 5, amplitude=0.02)
    got = []
    for own in (True, False):
        if not own:
            monkeypatch.undo()
        I = Interp(nx, ny, TWO_PI, TWO_PI, 0.8, 9.81, M)
        got.append((I.inverse_dtn(eta, v, 4), len(I.plan["inv_iter"])))
    assert rel(got[0][0], got[1][0]) < 1e-13
    assert got[0][1] == got[1][1] + (1 if M >= 2 else 0)
