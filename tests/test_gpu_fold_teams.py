"""The last level's G task on fold teams of every size class (FP64): one slot of a
wavefront, odd teams with shadow lanes, whole wavefronts, and the largest (ny = 640:
960 threads), against the oracle and against a batch, which runs it on plain
teams."""
import math

import numpy as np
import pytest

from oracle.hos import Grid, HOSModel
from paper_2608_25203_amd.inputs import random_band_fields

pytestmark = pytest.mark.gpu
TWO_PI = 2 * math.pi


@pytest.mark.parametrize("ny,M", [(32, 3), (48, 4), (64, 5), (80, 3), (96, 2), (160, 4), (320, 3), (384, 3), (512, 3),
                                  (640, 3), (640, 5), (768, 3)])
def test_fold_teams_match_oracle_and_plain_teams(ny, M):
    """The bars of test_gpu_parity.py (1e-10) and test_gpu_batch.py (1e-12)."""
    import torch

    from paper_2608_25203_amd.zk import Batch, Solver

    nx = 32
    Lx, Ly = TWO_PI * nx / 32, TWO_PI * ny / 32
    eta, psi = random_band_fields(nx, ny, 30 + M, 9, amplitude=0.02)
    s = Solver(nx, ny, Lx, Ly, 0.8, 9.81, M)
    e, p = torch.from_numpy(eta.copy()).cuda(), torch.from_numpy(psi.copy()).cuda()
    m = HOSModel(Grid(nx, ny, Lx, Ly, 0.8), M)
    ref = m.dtn(eta, psi)
    assert np.max(np.abs(s.dtn(e, p).cpu().numpy() - ref)) < 1e-10 * np.max(np.abs(ref))
    s.step(e, p, 0.002, 1)
    b = Batch([dict(nx=nx, ny=ny, Lx=Lx, Ly=Ly, depth=0.8, M=M)], g=9.81, precision=64)
    eb, pb = torch.from_numpy(eta.copy()).cuda(), torch.from_numpy(psi.copy()).cuda()
    b.set_fields([eb], [pb])
    b.step(0.002, 1)
    for x, y in ((e, eb), (p, pb)):
        assert float((x - y).abs().max()) < 1e-12 * float(y.abs().max())
