"""The phase recursion against the FP64 oracle at the edges of the step
schedule's range: radii of 2 to 7 pairs +-v per lane, exactly full lanes and
remainders, the smallest W, and a mean bispectrum that is zero for some w
(solve_in_steps says which of these run in steps and which in units)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import phase_rms, say

pytestmark = pytest.mark.gpu

# Both sides work in FP64 from the same float32 inputs.  A phasor is the unit of
# a sum of coherent samples, so its error is a few 2^-53 beyond that of the
# phasors it reads; along a chain of about 1000 steps that adds up to less
# than 1000 x 20 x 2^-53 = 2e-12 rad.
TOL = 2e-12


@pytest.mark.parametrize("N,u_cut,R", [(128, 63, 12), (128, 63, 9), (128, 63, 1), (128, 20, 12), (128, 3, 2),
                                       (64, 31, 12), (64, 31, 11), (64, 31, 8), (64, 2, 1)])
def test_phase_steps_against_the_oracle(N, u_cut, R):
    import torch
    import paper_1701_00581_amd as nv
    p = nv.default_params(N, u_cut=u_cut, v_radius=R)
    Wset, S, woff = oracle.bispectrum_set(u_cut, R)
    rng = np.random.default_rng(17 + N + u_cut + R)
    P = 3
    B = np.zeros((P, len(S)), np.complex128)
    M = np.zeros((P, 2), np.complex128)
    ix = lambda a, b: (b % N) * N + a % N  # noqa: E731
    for k in range(P):
        phi = rng.uniform(-np.pi, np.pi, N * N)
        phi[ix(-Wset[:, 0], -Wset[:, 1])] = -phi[ix(Wset[:, 0], Wset[:, 1])]
        wx, wy, vx, vy = S.T
        arg = phi[ix(wx - vx, wy - vy)] + phi[ix(vx, vy)] - phi[ix(wx, wy)]
        B[k] = (1 + 9 * rng.random(len(S))) * np.exp(1j * (arg + 0.3 * rng.standard_normal(len(S))))
        M[k] = 2 * np.exp(1j * phi[[1, N]])
    B[1, woff[len(Wset) - 2]:woff[len(Wset) - 1]] = 0      # a w whose sum is 0 gets the phasor 1
    M[2, 1] = 0
    B = B.astype(np.complex64)
    s = nv.Session(p, N, N + (P - 1) * p.stride, 1)
    assert s.info.patches == P and s.info.s_count == len(S)
    s.bispec.copy_(torch.from_numpy(np.ascontiguousarray(B).view(np.float32).reshape(P, len(S), 2)))
    s.mean_spec.copy_(torch.from_numpy(M.astype(np.complex64).view(np.float32).reshape(P, 2, 2)))
    s.power.fill_(1.0)
    stf = torch.ones(N, N, dtype=torch.float64, device="cuda")
    for _ in range(2):                                     # a second launch finds LDS in use
        s.phasor.fill_(float("nan"))
        s.solve(stf)
    e = s.phasor.cpu().numpy()
    e = e[..., 0] + 1j * e[..., 1]
    for k in range(P):
        M32 = M[k].astype(np.complex64)
        ref = oracle.phase_recursion(B[k].astype(np.complex128), M32[0], M32[1], Wset, S, woff, N)
        rms, worst = phase_rms(e[k], ref)
        say(f"N {N} u_cut {u_cut} R {R} patch {k}: rms {rms:.1e} worst {worst:.1e}")
        assert rms <= TOL and np.max(np.abs(np.abs(e[k]) - 1)) < 1e-12
    assert torch.equal(s.amp, torch.ones_like(s.amp))
    s.close()


def test_batch_of_both_kinds_equals_alone():
    """A batch whose bursts hold fewer and more patches than the card has CUs
    (256): each burst's image is that of the same burst alone, bit for bit."""
    import torch
    import paper_1701_00581_amd as nv
    p = nv.default_params(64, v_radius=4, stride=32)
    g = torch.Generator(device="cuda").manual_seed(3)
    shapes = [(4, 96, 128), (3, 32 * 17, 32 * 19), (2, 32 * 17, 32 * 17), (3, 64, 64), (2, 32 * 18, 32 * 17)]
    assert [nv.nvsm_plan(p, h, w, f).patches for f, h, w in shapes] == [6, 16 * 18, 256, 1, 17 * 16]
    bursts = []
    for f, h, w in shapes:
        fr = 1000 * (1 + 0.2 * torch.rand(f, h, w, device="cuda", generator=g))
        bursts.append((fr, torch.ones(64, 64, dtype=torch.float64, device="cuda"), torch.zeros(h, w, device="cuda")))
    ctx = nv.nvsm_create(0)
    ws = torch.empty(nv.nvsm_batch_plan(p, shapes)[1], dtype=torch.uint8, device="cuda")
    nv.nvsm_reconstruct_batch(ctx, p, bursts, ws)
    together = [b[2].clone() for b in bursts]
    for (fr, st, out), ref in zip(bursts, together):
        out.zero_()
        nv.nvsm_reconstruct(ctx, p, fr, st, out, ws)
        assert torch.equal(out, ref)
    torch.cuda.synchronize()
    nv.nvsm_destroy(ctx)


@pytest.mark.parametrize("N,u_cut,R,spike", [(128, 63, 12, 1), (128, 40, 9, 1), (64, 31, 8, 1e7), (64, 20, 12, 1e3),
                                             (64, 5, 4, 1), (64, 2, 1, 1)])
def test_least_squares_pairs_against_the_oracle(N, u_cut, R, spike):
    """The least-squares steps with pairs over the lanes (k_lsq_pairs): 2 and 4
    pairs per lane, W shorter than a round, and a sample that outweighs the
    others (its adds take the full conversion)."""
    import torch
    import paper_1701_00581_amd as nv
    p = nv.default_params(N, u_cut=u_cut, v_radius=R, phase_method=1, lsq_iters=3)
    Wset, S, woff = oracle.bispectrum_set(u_cut, R)
    rng = np.random.default_rng(N + u_cut + R)
    phi = rng.uniform(-np.pi, np.pi, N * N)
    ix = lambda a, b: (b % N) * N + a % N  # noqa: E731
    phi[ix(-Wset[:, 0], -Wset[:, 1])] = -phi[ix(Wset[:, 0], Wset[:, 1])]
    wx, wy, vx, vy = S.T
    arg = phi[ix(wx - vx, wy - vy)] + phi[ix(vx, vy)] - phi[ix(wx, wy)]
    B = (1 + 9 * rng.random(len(S))) * np.exp(1j * (arg + 0.5 * rng.standard_normal(len(S))))
    B[len(S) // 2] *= spike
    B = B.astype(np.complex64)
    M = (2 * np.exp(1j * phi[[1, N]])).astype(np.complex64)
    s = nv.Session(p, N, N, 1)
    s.bispec.copy_(torch.from_numpy(B.view(np.float32).reshape(1, len(S), 2)))
    s.mean_spec.copy_(torch.from_numpy(M.view(np.float32).reshape(1, 2, 2)))
    s.power.fill_(1.0)
    s.solve(torch.ones(N, N, dtype=torch.float64, device="cuda"))
    e = s.phasor.cpu().numpy()[0]
    e = e[..., 0] + 1j * e[..., 1]
    first = s.phasor.clone()
    s.solve(torch.ones(N, N, dtype=torch.float64, device="cuda"))
    assert torch.equal(first, s.phasor)                    # integer adds: repeatable
    s.close()
    B64 = B.astype(np.complex128)
    ref = oracle.phase_recursion(B64, M[0], M[1], Wset, S, woff, N)
    ref = oracle.phase_least_squares(B64, ref, Wset, S, woff, 3)
    rms, worst = phase_rms(e, ref)
    say(f"lsq N {N} u_cut {u_cut} R {R}: rms {rms:.1e} worst {worst:.1e}")
    # an add is off by half a unit, s1 2^-62 (s1 = sum |Re B| + |Im B|); a sum
    # has at most a few hundred adds and |g| at least 1 here, and a step at
    # most doubles what the one before left
    s1 = float(np.abs(B64.real).sum() + np.abs(B64.imag).sum())
    assert worst <= 8 * (300 * s1 * 2.0 ** -62 + TOL)
