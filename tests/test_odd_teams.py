"""Teams of 3 2^k and 5 2^k threads (axes with a factor 3 or 5): their pass
plan on the CPU, and on the GPU every compiled team shape of such axes."""
import math
import os
import re

import numpy as np
import pytest

import test_fft_model as F

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_25203_amd", "csrc")
ODD = [3 * 2 ** k for k in range(1, 9)] + [5 * 2 ** k for k in range(1, 8)]


def pass_radix(T, E, rem):
    return 3 if rem % 3 == 0 else 5 if rem % 5 == 0 else POW2_RADIX(T, E, rem)


POW2_RADIX = F.pass_radix


@pytest.mark.parametrize("E", [2, 3])
@pytest.mark.parametrize("T", ODD)
def test_odd_team_fft_matches_numpy(monkeypatch, T, E):
    """One radix-3 or radix-5 pass after the first, then the plan of a
    power-of-two team: the model of test_fft_model.py with the kernels'
    pass_radix, against numpy at that file's bar."""
    monkeypatch.setattr(F, "pass_radix", pass_radix)
    F.test_team_fft_forms_match_numpy(T, E)


def test_further_unit_parts_are_current(tmp_path):
    """The further parts of the generated units, and the build's list of them."""
    import shutil
    import subprocess
    import sys

    from paper_2608_25203_amd.build import HIP_UNITS

    shutil.copy(os.path.join(CSRC, "gen_batch_units.py"), tmp_path)
    subprocess.run([sys.executable, str(tmp_path / "gen_batch_units.py")], check=True)
    made = sorted(f for f in os.listdir(tmp_path) if f.endswith(".hip"))
    assert made == sorted(f for f in os.listdir(CSRC) if re.match(r"zk_batch_(row|col)_", f))
    assert made == sorted(u for u in HIP_UNITS if u.startswith("zk_batch_"))
    for f in made:
        assert (tmp_path / f).read_text() == open(os.path.join(CSRC, f)).read(), f


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(48, 12), (96, 24), (192, 320), (80, 40), (160, 384), (640, 20)])
def test_odd_axis_team_shapes(nx, ny):
    """Each axis with teams of n / 2 threads (the FP64 default) and with the
    power-of-two team of its radix-9 or radix-15 step (FP32's): the RHS against
    the oracle, FP64 at 1e-10 and FP32 at 2e-5 (the bars of test_gpu_parity.py)."""
    import torch

    from oracle.hos import Grid, HOSModel
    from paper_2608_25203_amd.inputs import random_band_fields
    from paper_2608_25203_amd.zk import Solver

    M, Lx, Ly, h = 3, 2.0, 2.0 * ny / nx, 0.6
    kmax = math.hypot(math.pi * nx / Lx, math.pi * ny / Ly)
    eta, psi = random_band_fields(nx, ny, 7, min(nx, ny) // 2 - 1, amplitude=0.1 / kmax)
    a0, b0 = HOSModel(Grid(nx, ny, Lx, Ly, h), M).rhs(eta, psi)
    e, p = (torch.tensor(x, dtype=torch.float64, device="cuda") for x in (eta, psi))
    for prec, tol in ((64, 1e-10), (32, 2e-5)):
        s = Solver(nx, ny, Lx, Ly, h, 9.81, M, precision=prec)
        for old in (False, True) if prec == 64 else (True,):
            for row, n in ((1, nx), (0, ny)):
                f = 3 if n % 3 == 0 else 5
                for pad in (1, 0):
                    N = 3 * n // 2 if pad else n
                    s.set_team_shape(row, pad, N // ((3 * f) if pad else (2 * f)) if old else n // 2)
            print(" ", prec, s.team_shapes(), flush=True)
            for got, ref in zip(s.rhs(e, p), (a0, b0)):
                assert np.max(np.abs(got.cpu().numpy() - ref)) < tol * np.max(np.abs(ref))
