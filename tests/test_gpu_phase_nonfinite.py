"""The phase recursion in steps (k_phase) with samples or seeds that are not
finite: the damage stays with the frequencies that use them."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _recursion(B, M, Wset, S, woff, N):
    """oracle.phase_recursion with the kernel's rule: a sum whose square is
    infinite, or a seed that is, gives no phasor (NaN), which counts as 0 where
    it is read, and a sum that is not a number gives the phasor 1."""
    E = np.zeros((N, N), np.complex128)
    out = np.zeros(len(Wset), np.complex128)
    for i, (x, y) in enumerate(Wset):
        if i < 2:
            v = M[i] / abs(M[i]) if np.isfinite(M[i]) else complex(np.nan, np.nan)
        else:
            s = S[woff[i]:woff[i + 1]]
            p = E[(y - s[:, 3]) % N, (x - s[:, 2]) % N] * E[s[:, 3] % N, s[:, 2] % N]
            t = B[woff[i]:woff[i + 1]]
            zx = np.sum(p.real * t.real + p.imag * t.imag)
            zy = np.sum(p.imag * t.real - p.real * t.imag)
            n = zx * zx + zy * zy
            v = complex(np.nan, np.nan) if n == np.inf else complex(zx, zy) / np.sqrt(n) if n > 0 else 1.0
        out[i] = v
        e = v if np.isfinite(v) else 0.0
        E[y % N, x % N], E[-y % N, -x % N] = e, np.conj(e)
    return out


@pytest.mark.parametrize("N,u_cut,R", [(64, 31, 6), (64, 31, 2), (128, 63, 10)])
@pytest.mark.parametrize("where", ["inner sample", "outer sample", "seed"])
def test_nonfinite_inputs_stay_contained(N, u_cut, R, where):
    import torch
    import paper_1701_00581_amd as nv
    p = nv.default_params(N, u_cut=u_cut, v_radius=R)
    Wset, S, woff = oracle.bispectrum_set(u_cut, R)
    rng = np.random.default_rng(N + R)
    ix = lambda a, b: (b % N) * N + a % N  # noqa: E731
    phi = rng.uniform(-np.pi, np.pi, N * N)
    phi[ix(-Wset[:, 0], -Wset[:, 1])] = -phi[ix(Wset[:, 0], Wset[:, 1])]
    wx, wy, vx, vy = S.T
    arg = phi[ix(wx - vx, wy - vy)] + phi[ix(vx, vy)] - phi[ix(wx, wy)]
    B = ((1 + 9 * rng.random(len(S))) * np.exp(1j * (arg + 0.3 * rng.standard_normal(len(S))))).astype(np.complex64)
    M = (2 * np.exp(1j * phi[[1, N]])).astype(np.complex64)
    inner = int((Wset[:, 0] ** 2 + Wset[:, 1] ** 2 <= R * R).sum())
    if where == "seed":
        M[0] = complex(np.inf, 1)
    else:
        w = inner - 2 if where == "inner sample" else (inner + len(Wset)) // 2
        t = woff[w] + (woff[w + 1] - woff[w]) // 2
        B[t] = complex(np.inf, B[t].imag)          # one sample past float32
    s = nv.Session(p, N, N, 1)
    s.bispec.copy_(torch.from_numpy(B.view(np.float32).reshape(1, len(S), 2)))
    s.mean_spec.copy_(torch.from_numpy(M.view(np.float32).reshape(1, 2, 2)))
    s.power.fill_(1.0)
    st = torch.ones(N, N, dtype=torch.float64, device="cuda")
    s.solve(st)
    first = s.phasor.clone()
    for _ in range(3):
        s.solve(st)
        assert torch.equal(torch.nan_to_num(first, nan=9.0), torch.nan_to_num(s.phasor, nan=9.0))
    s.close()
    e = first.cpu().numpy()[0]
    e = e[:, 0] + 1j * e[:, 1]
    with np.errstate(all="ignore"):
        ref = _recursion(B.astype(np.complex128), M.astype(np.complex128), Wset, S, woff, N)
    bad = ~np.isfinite(ref)
    assert 1 <= bad.sum() <= 2 and not np.isfinite(e[bad]).any()
    # 2e-12 rad is about 1000 links of 20 roundings of 2^-53; 100 times that for the
    # worst of the w, whose samples may nearly cancel beside a missing one
    assert np.isfinite(e[~bad]).all() and np.abs(np.angle(e[~bad] * np.conj(ref[~bad]))).max() <= 2e-10
