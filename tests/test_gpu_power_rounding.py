"""Rounding of the power spectrum's sum over the frames alone: the mean power
of one frame group against the same stored spectra in FP64, with few patches
(sums formed after the ingest) and many (formed by it)."""
import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,side", [(64, 2), (64, 12), (128, 2), (128, 12)])
def test_power_sum_rounds_once_a_frame(N, side):
    import torch
    import paper_1701_00581_amd as nv
    F = 16                                     # one group; a mean over 16 rounds nothing
    p = nv.default_params(N, v_radius=2)
    L = N + (side - 1) * N // 2
    s = nv.Session(p, L, L, F)
    P, rows = s.info.patches, N // 2 + 16
    assert P == side * side
    g = torch.Generator(device="cuda").manual_seed(N + side)
    s.accumulate(1000 + 3000 * torch.rand(F, L, L, device="cuda", generator=g), with_bispectrum=False)
    rec = s.ws_acc[:P * F * rows * N * 8].view(torch.float32).view(P, F, rows, N, 2)[:, :, 16:].cpu().numpy()
    got = s.power[:, :N // 2].cpu().numpy()
    s.close()
    x, y = rec[..., 0], rec[..., 1]
    exact = (x.astype(np.float64) ** 2 + y.astype(np.float64) ** 2).mean(1)
    t = np.zeros_like(got)
    for f in range(F):                         # |I|^2 (a product, a fused multiply-add), then one addition
        t = t + (x[:, f].astype(np.float64) ** 2 + y[:, f] * y[:, f]).astype(np.float32)
    t /= F
    rms = lambda z: float(np.sqrt(np.mean((z[:, 1:] / exact[:, 1:] - 1) ** 2)))  # noqa: E731  (row 0 holds u = 0)
    say(f"N {N} {P} patches: kernel {rms(got):.3e}, one rounding a frame {rms(t):.3e} rms over {got[:, 1:].size}")
    # over at least 7000 values an rms is known to 1/sqrt(2 x 7000) = 0.85 %
    assert got[:, 1:].size > 7000 and rms(got) <= 1.04 * rms(t)
