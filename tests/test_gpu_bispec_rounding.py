"""Arithmetic of the bispectrum terms alone: the FP32 products of the stored
spectra of one frame against the same products in FP64.  (The mean over the
frames and the image inherit this error, and a frequency whose samples nearly
cancel passes it on enlarged.)"""
import numpy as np
import pytest

import oracle
from gpu_helpers import say

pytestmark = pytest.mark.gpu


def _fma(a, b, c):
    """float32 a b + c, rounded once (the product is exact in float64)."""
    return (a.astype(np.float64) * b + c).astype(np.float32)


@pytest.mark.parametrize("N,R", [(64, 8), (64, 12), (128, 10)])
def test_terms_round_no_more_than_complex_products(N, R):
    import torch
    import paper_1701_00581_amd as nv
    p = nv.default_params(N, v_radius=R)
    Wset, S, _ = oracle.bispectrum_set(p.u_cut, R)
    s = nv.Session(p, N, 2 * N, 1)
    P, rows = s.info.patches, N // 2 + 16
    g = torch.Generator(device="cuda").manual_seed(N + R)
    s.accumulate(1000 + 3000 * torch.rand(1, N, 2 * N, device="cuda", generator=g))
    rec = s.ws_acc[:P * rows * N * 8].view(torch.float32).view(P, rows, N, 2).cpu().numpy()   # rows -16 .. N/2 - 1
    got = s.bispec.cpu().numpy()
    s.close()
    wx, wy, vx, vy = S.T
    at = lambda x, y: (slice(None), y + 16, x % N)  # noqa: E731
    a, v, w = rec[at(wx - vx, wy - vy)], rec[at(vx, vy)], rec[at(wx, wy)]
    cplx = lambda z: z[..., 0].astype(np.float64) + 1j * z[..., 1]  # noqa: E731
    exact = cplx(a) * cplx(v) * np.conj(cplx(w))
    # p = I(w - v) I(v), t = p conj I(w): a product and a fused multiply-add
    # for each part of each of the two, eight roundings a term
    pr = _fma(v[..., 0], a[..., 0], -v[..., 1] * a[..., 1])
    pi = _fma(v[..., 1], a[..., 0], v[..., 0] * a[..., 1])
    t = _fma(pr, w[..., 0], pi * w[..., 1]) + 1j * _fma(pi, w[..., 0], -pr * w[..., 1])
    rms = lambda z: float(np.sqrt(np.mean((np.abs(z - exact) / np.abs(exact)) ** 2)))  # noqa: E731
    kernel, eight = rms(cplx(got)), rms(t)
    say(f"N {N} R {R}: kernel {kernel:.3e}, two complex products {eight:.3e} of |term| rms over {exact.size} terms")
    # over at least 10^5 terms an rms is known to 1/sqrt(2 10^5) = 0.3 %
    assert exact.size > 1e5 and kernel <= 1.01 * eight
