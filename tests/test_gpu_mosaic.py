"""The mosaic's four-pixel and one-pixel forms against the oracle's, where
they can differ: widths and strides that are and are not multiples of 4, an
unaligned subimage buffer, and images narrower and wider than a workgroup's
pixels."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,stride,shift", [(100, 128, 32, 0), (97, 131, 32, 0), (97, 130, 31, 0), (65, 1100, 32, 0),
                                              (65, 1102, 32, 0), (70, 128, 32, 1), (64, 64, 64, 0)])
def test_mosaic_forms(H, W, stride, shift):
    import torch
    import paper_1701_00581_amd as nv
    N = 64
    p = nv.default_params(N, v_radius=2, u_cut=5, stride=stride)
    ys, xs = oracle.tiling(H, W, N, stride)
    P, nW = len(ys) * len(xs), len(oracle.frequency_half_disk(5))
    mu = torch.rand(P, device="cuda", generator=torch.Generator(device="cuda").manual_seed(5)) + 1
    buf = torch.empty(P * N * N + 4, device="cuda")[shift:shift + P * N * N]
    out = torch.full((H, W), float("nan"), device="cuda")
    ctx = nv.nvsm_create(0)
    nv.nvsm_synthesize(ctx, p, H, W, torch.zeros(P, nW, dtype=torch.float64, device="cuda"),
                       torch.ones(P, nW, 2, dtype=torch.float64, device="cuda"), mu, buf, out)
    torch.cuda.synchronize()
    nv.nvsm_destroy(ctx)
    sub = buf.double().cpu().numpy().reshape(len(ys), len(xs), N, N)
    ref = oracle.mosaic(sub, ys, xs, H, W, 1)
    got = out.cpu().numpy()
    on = oracle.mosaic(np.ones_like(sub) * oracle.window2d(N, 1), ys, xs, H, W, 1) > 0   # the taper sum is above its floor
    # at most 9 terms and the taper's sums in float32, relative to a sum of
    # the same sign: 16 roundings of 2^-24; the taper sum near its floor of
    # 1e-3 is itself a sum of terms of at most 1, with 2 2^-24 of error
    assert np.isfinite(got).all() and np.max(np.abs(got - ref)[on] / 2) <= 16 * 2.0 ** -24 + 4 * 2.0 ** -24 / 1e-3
