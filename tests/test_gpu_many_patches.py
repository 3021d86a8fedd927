"""A burst of more patches than a one-dimensional grid of the passes over a
patch's parts can number (1.87 million at N = 64): every patch is written, with
the values it has in a small burst."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noise_bias", [0, 2])
def test_every_patch_of_a_very_large_burst_is_written(noise_bias):
    import torch
    import paper_1701_00581_amd as nv
    N, stride, side = 64, 4, 1366
    p = nv.default_params(N, v_radius=2, u_cut=4, stride=stride, noise_bias=noise_bias, photons_per_adu=2.0)
    L = N + (side - 1) * stride
    info = nv.nvsm_plan(p, L, L, 1)
    P = info.patches
    assert P == side * side and P * 9 * 256 > 1 << 32
    if torch.cuda.mem_get_info()[0] < info.ws_accumulate + P * N * N * 4 + (8 << 30):
        pytest.skip("not enough device memory")
    frame = 1000 * torch.rand(1, L, L, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    ctx = nv.nvsm_create(0)

    def accumulate(fr, patches, ws_bytes):
        power = torch.full((patches, N, N), float("nan"), device="cuda")
        mean = torch.full((patches, 2, 2), float("nan"), device="cuda")
        mu = torch.full((patches,), float("nan"), device="cuda")
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
        nv.nvsm_accumulate(ctx, p, fr, power, mean, mu, None, ws)
        torch.cuda.synchronize()
        return power, mean, mu

    power, mean, mu = accumulate(frame, P, info.ws_accumulate)
    for t in (power[:, 0, 1], power[:, N - 1, N - 1], power[:, N // 2, 0], mean[:, 1, 1], mu):
        assert not torch.isnan(t).any()
    for k in (0, 1, P // 2, P - 2, P - 1):
        y, x = k // side * stride, k % side * stride
        one = accumulate(frame[:, y:y + N, x:x + N].contiguous(), 1, nv.nvsm_plan(p, N, N, 1).ws_accumulate)
        for a, b in zip((power, mean, mu), one):
            assert torch.equal(a[k:k + 1], b)
    nv.nvsm_destroy(ctx)
    del power, mean, mu
    torch.cuda.empty_cache()


@pytest.mark.parametrize("N,dtype", [(64, "float32"), (128, "uint16")])
def test_parts_of_a_patch_do_not_change_its_sums(N, dtype):
    """The passes over the frame groups split a patch by the number of patches
    (one entry a thread, fewer workgroups above 4096 / parts): a patch's power,
    means and photon-noise terms are the same for 1, 36 and 2025 of them."""
    import torch
    import paper_1701_00581_amd as nv
    F, stride = 23, N // 2
    for noise_bias in (0, 2):
        p = nv.default_params(N, v_radius=2, u_cut=4, noise_bias=noise_bias, photons_per_adu=2.0)
        L = lambda side: N + (side - 1) * stride  # noqa: E731
        g = torch.Generator(device="cuda").manual_seed(N)
        fr = (100 + 3000 * torch.rand(F, L(45), L(45), device="cuda", generator=g)).to(getattr(torch, dtype))
        ref = None
        for side in (45, 6, 1):
            s = nv.Session(p, L(side), L(side), F)
            s.accumulate(fr[:, :L(side), :L(side)].contiguous())
            rows = [y * side + x for y in range(min(side, 6)) for x in range(min(side, 6))]
            got = [t[rows].clone() for t in (s.power, s.mean_spec, s.mu, s.bispec)]
            s.close()
            ref = ref or got
            assert all(torch.equal(a[:len(rows)], b) for a, b in zip(ref, got))
