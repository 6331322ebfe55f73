"""The default base row teams of 256 and 1024 points (E = 4, FP64) against the
n / 2-thread teams: the depth lift and one DtN give the same fields."""
import math

import pytest

from paper_2608_25203_amd.inputs import random_band_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,E", [(256, 16, 4), (1024, 16, 4), (512, 16, 2)])
def test_base_row_default_matches_two_point_first_pass(nx, ny, E):
    """Both round FP64 transforms of at most 1024 points differently: 1e-12 of
    the largest value, a thousand roundings."""
    import torch

    from paper_2608_25203_amd.zk import Solver

    s = Solver(nx, ny, 2.0 * math.pi * nx / ny, 2.0 * math.pi, 0.6, 9.81, 2)
    eta, psi = (torch.from_numpy(f).cuda() for f in random_band_fields(nx, ny, 77, 5, amplitude=0.01))
    ys = [0.0, 0.25, 0.6]
    a = s.depth_velocity(eta, psi, ys), s.dtn(eta, psi)
    assert s.team_shapes()["row_base"] == (nx // E, E)
    s.set_team_shape(1, 0, nx // 2)
    b = s.depth_velocity(eta, psi, ys), s.dtn(eta, psi)
    for x, y in zip(a, b):
        assert float((x - y).abs().max()) <= 1e-12 * float(y.abs().max())
