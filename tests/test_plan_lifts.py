"""The sequences that step and lift in one launch (step_body_lift,
ab2_*_lift), executed literally by the numpy interpreter, against the oracle;
split lifts on small grids, merged ones above 2^18 points."""
import math

import pytest

from oracle.hos import Grid, HOSModel
from paper_2608_25203_amd.inputs import random_band_fields
from plan_interp import Interp
from test_host import rel

TWO_PI = 2 * math.pi


def run_fused(I, eta, psi, dt, nsteps, ab2):
    P = I._plan(dt)
    phys = [eta, psi, 0 * eta, 0 * eta]
    I.run(P["step_entry"], phys)
    for i in range(nsteps):
        name = ("ab2_first" if i == 0 else "ab2_body") if ab2 else "step_body"
        I.run(P[name + ("" if i + 1 == nsteps else "_lift") + str(i & 1)], phys)
    I.run(P["step_exit%d" % (nsteps & 1)], phys)
    return phys[2], phys[3]


@pytest.mark.parametrize("ab2", [False, True])
@pytest.mark.parametrize("nx,ny,M", [(32, 32, 1), (32, 32, 2), (32, 48, 3), (32, 32, 4), (48, 32, 5), (64, 1, 3),
                                     (32, 32, 8), (2048, 1, 3), (640, 512, 2), (1024, 320, 3)])
def test_fused_lift_sequences_match_oracle(nx, ny, M, ab2):
    """Three steps (both parities, the last without lifts); the same bar as
    the schedule checks of test_host.py (rounding of order-M sums, 1e-13)."""
    Lx, Ly = TWO_PI * nx / 32, (TWO_PI * ny / 32 if ny > 1 else 1.0)
    eta, psi = random_band_fields(nx, ny, 40 + M, 5, amplitude=0.02)
    I = Interp(nx, ny, Lx, Ly, 0.8, 9.81, M)
    m = HOSModel(Grid(nx, ny, Lx, Ly, 0.8), M)
    got = run_fused(I, eta, psi, 0.004, 3, ab2)
    ref = (m.step_ifab2 if ab2 else m.step)(eta, psi, 0.004, 3)
    for a, b in zip(got, ref):
        assert rel(a, b) < 1e-13


def test_tall_grid_splits_its_lifts():
    """Above 2^18 points but on rows of fewer than 512: the fused sequences
    of the split form, the bar as above."""
    nx, ny, M = 320, 1024, 2
    Lx, Ly = TWO_PI * nx / 32, TWO_PI * ny / 32
    eta, psi = random_band_fields(nx, ny, 45, 5, amplitude=0.02)
    I = Interp(nx, ny, Lx, Ly, 0.8, 9.81, M)
    m = HOSModel(Grid(nx, ny, Lx, Ly, 0.8), M)
    for a, b in zip(run_fused(I, eta, psi, 0.004, 2, False), m.step(eta, psi, 0.004, 2)):
        assert rel(a, b) < 1e-13
