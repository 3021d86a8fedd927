"""The phase recursion's kernel forms against the FP64 oracle with more patches
than the card has CUs: units of 2 and 4 samples per lane (k_solve), steps with
2 and 5 pairs +-v per lane (k_phase).  And batches: bursts of a few patches
between larger ones cost no more than the same bursts in another order."""
import numpy as np
import pytest

import oracle
from gpu_helpers import phase_rms, say

pytestmark = pytest.mark.gpu

# as in the test of the steps: about 1000 links of a few roundings of 2^-53 each
TOL = 2e-12


def _inputs(rng, N, Wset, S):
    ix = lambda a, b: (b % N) * N + a % N  # noqa: E731
    phi = rng.uniform(-np.pi, np.pi, N * N)
    phi[ix(-Wset[:, 0], -Wset[:, 1])] = -phi[ix(Wset[:, 0], Wset[:, 1])]
    wx, wy, vx, vy = S.T
    arg = phi[ix(wx - vx, wy - vy)] + phi[ix(vx, vy)] - phi[ix(wx, wy)]
    B = (1 + 9 * rng.random(len(S))) * np.exp(1j * (arg + 0.3 * rng.standard_normal(len(S))))
    return B.astype(np.complex64), (2 * np.exp(1j * phi[[1, N]])).astype(np.complex64)


@pytest.mark.parametrize("N,u_cut,R", [
    (64, 31, 1), (64, 31, 6), (64, 6, 3), (128, 63, 10), (128, 60, 10),                     # steps
    (64, 31, 7), (64, 31, 9), (64, 31, 10), (64, 31, 12), (128, 63, 7), (128, 63, 9), (128, 59, 10), (128, 63, 12)])
def test_recursion_forms_against_the_oracle(N, u_cut, R):
    import torch
    import paper_1701_00581_amd as nv
    P = 258                                                # past one workgroup per CU
    p = nv.default_params(N, u_cut=u_cut, v_radius=R)
    Wset, S, woff = oracle.bispectrum_set(u_cut, R)
    rng = np.random.default_rng(N + u_cut + R)
    B, M = zip(*(_inputs(rng, N, Wset, S) for _ in range(2)))
    s = nv.Session(p, N, N + (P - 1) * p.stride, 1)
    assert s.info.patches == P and s.info.s_count == len(S)
    bd = torch.stack([torch.from_numpy(b.view(np.float32).reshape(-1, 2)) for b in B]).cuda()
    md = torch.stack([torch.from_numpy(m.view(np.float32).reshape(2, 2)) for m in M]).cuda()
    for k in range(2):                                     # two inputs, in turn
        s.bispec[k::2] = bd[k]
        s.mean_spec[k::2] = md[k]
    s.power.fill_(1.0)
    s.phasor.fill_(float("nan"))
    s.solve(torch.ones(N, N, dtype=torch.float64, device="cuda"))
    e = s.phasor
    assert all(torch.equal(e[k::2], e[k].expand_as(e[k::2])) for k in range(2))   # every patch as the first two
    for k in range(2):
        got = e[k].cpu().numpy()
        got = got[..., 0] + 1j * got[..., 1]
        ref = oracle.phase_recursion(B[k].astype(np.complex128), M[k][0], M[k][1], Wset, S, woff, N)
        rms, worst = phase_rms(got, ref)
        say(f"N {N} u_cut {u_cut} R {R} input {k}: rms {rms:.1e} worst {worst:.1e}")
        assert rms <= TOL and np.max(np.abs(np.abs(got) - 1)) < 1e-12
    s.close()


@pytest.mark.parametrize("R", [4, 8])
def test_order_of_a_batch_costs_nothing(R):
    """One-patch bursts between bursts of 300: the solve of the group is one
    launch whatever their order, so it takes the time of the same bursts
    sorted (a launch for each run of a kind took three times that)."""
    import torch
    import paper_1701_00581_amd as nv
    N, F = 64, 2
    p = nv.default_params(N, v_radius=R)
    small, large = (F, 64, 64), (F, 16 * 32, 21 * 32)
    assert [nv.nvsm_plan(p, h, w, f).patches for f, h, w in (small, large)] == [1, 300]
    g = torch.Generator(device="cuda").manual_seed(R)
    st = torch.ones(N, N, dtype=torch.float64, device="cuda")
    make = lambda f, h, w: (1000 + 200 * torch.rand(f, h, w, device="cuda", generator=g), st,  # noqa: E731
                            torch.empty(h, w, device="cuda"))
    apart = [make(*c) for c in [small] * 8 + [large] * 8]
    mixed = [b for pair in zip(apart[:8], apart[8:]) for b in pair]
    ctx = nv.nvsm_create(0)
    ws = torch.empty(nv.nvsm_batch_plan(p, [tuple(b[0].shape) for b in apart])[1], dtype=torch.uint8, device="cuda")
    nv.nvsm_profile_enable(ctx, True)

    def solve_ms(bursts):
        best = float("inf")
        for _ in range(5):
            nv.nvsm_profile_read(ctx)
            nv.nvsm_reconstruct_batch(ctx, p, bursts, ws)
            torch.cuda.synchronize()
            best = min(best, nv.nvsm_profile_read(ctx)["solve"][0])
        return best

    images = []
    times = []
    for bursts in (apart, mixed, apart, mixed):
        times.append(solve_ms(bursts))
        images.append([b[2].clone() for b in apart])
    say(f"R {R}: solve of the sorted batch {min(times[::2]):.3f} ms, alternating {min(times[1::2]):.3f} ms")
    assert min(times[1::2]) <= 1.5 * min(times[::2])
    assert all(torch.equal(a, b) for a, b in zip(images[0], images[1]))
    nv.nvsm_destroy(ctx)


@pytest.mark.parametrize("N,u_cut,R", [(128, 63, 10), (64, 31, 9), (64, 31, 10), (64, 31, 11)])
def test_least_squares_with_three_pairs_per_lane(N, u_cut, R):
    """The least-squares steps at 2, 3 and 4 pairs per lane on either side of
    each change, against the oracle."""
    import torch
    import paper_1701_00581_amd as nv
    p = nv.default_params(N, u_cut=u_cut, v_radius=R, phase_method=1, lsq_iters=2)
    Wset, S, woff = oracle.bispectrum_set(u_cut, R)
    B, M = _inputs(np.random.default_rng(5 + N + R), N, Wset, S)
    s = nv.Session(p, N, N, 1)
    s.bispec.copy_(torch.from_numpy(B.view(np.float32).reshape(1, len(S), 2)))
    s.mean_spec.copy_(torch.from_numpy(M.view(np.float32).reshape(1, 2, 2)))
    s.power.fill_(1.0)
    s.solve(torch.ones(N, N, dtype=torch.float64, device="cuda"))
    e = s.phasor.cpu().numpy()[0]
    s.close()
    B64 = B.astype(np.complex128)
    ref = oracle.phase_recursion(B64, M[0], M[1], Wset, S, woff, N)
    ref = oracle.phase_least_squares(B64, ref, Wset, S, woff, 2)
    rms, worst = phase_rms(e[..., 0] + 1j * e[..., 1], ref)
    say(f"lsq N {N} R {R}: rms {rms:.1e} worst {worst:.1e}")
    # as in the test of the pairs: adds off by half a unit of s1 2^-62, a few
    # hundred to a sum of modulus at least 1, doubled by each of two steps
    s1 = float(np.abs(B64.real).sum() + np.abs(B64.imag).sum())
    assert worst <= 4 * (300 * s1 * 2.0 ** -62 + TOL)
