"""The weight-gradient kernels where a wavefront walks more than one strip."""
import numpy as np
import pytest

from oracle import cnn as C
from paper_2608_25203_amd.inputs import cnn_init_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,W", [(1100, 5, 64), (260, 9, 256)])
def test_gradient_of_more_strips_than_wavefronts(B, H, W):
    """B (W / 64) strips in two bands each: more than the 2048 wavefronts of
    the 256 blocks, while a half of the batch has at most one a wavefront.  The
    gradient is the mean of its halves': halving the batch scales every bf16
    operand by a power of two, so the two sides differ by the order of FP32 sums
    alone (a few hundred roundings of 6e-8 on sums that cancel to about their
    root mean square: 1e-4 of each tensor's largest value is a wide bound; one
    strip of 2200 is about 1 / sqrt(2200) of such a sum)."""
    import torch

    from paper_2608_25203_amd.zk import Net

    p32 = C.flatten([p * 2.0 if p.ndim == 4 else p for p in cnn_init_params(11)]).astype(np.float32)
    x = np.random.default_rng(12).standard_normal((B, 4, H, W))
    s = torch.tensor(x, dtype=torch.float32, device="cuda")
    net = Net(B * H * W)
    net.set_params(p32)
    loss, g = net.gradient(s, 2)
    parts = [net.gradient(h.contiguous(), 2) for h in (s[:B // 2], s[B // 2:])]
    assert abs(loss - 0.5 * (parts[0][0] + parts[1][0])) < 1e-9 * abs(loss)
    whole = C.unflatten(g.astype(np.float64))
    halves = C.unflatten(0.5 * (parts[0][1].astype(np.float64) + parts[1][1]))
    for a, b in zip(whole, halves):
        assert np.max(np.abs(a - b)) < 1e-4 * np.max(np.abs(b))
