"""The mosaic of a batch of images of very different widths: each image's
pixels are those of the image alone, and a wide image leaves no idle work
beside narrow ones."""
import pytest

pytestmark = pytest.mark.gpu


def _run(shapes, stride, reps=1):
    import torch
    import paper_1701_00581_amd as nv
    N = 64
    p = nv.default_params(N, v_radius=2, u_cut=4, stride=stride)
    g = torch.Generator(device="cuda").manual_seed(len(shapes))
    st = torch.ones(N, N, dtype=torch.float64, device="cuda")
    bursts = [(1000 + torch.rand(f, h, w, device="cuda", generator=g), st,
               torch.full((h, w), float("nan"), device="cuda")) for f, h, w in shapes]
    ctx = nv.nvsm_create(0)
    ws = torch.empty(nv.nvsm_batch_plan(p, shapes)[1], dtype=torch.uint8, device="cuda")
    nv.nvsm_profile_enable(ctx, True)
    best = float("inf")
    for _ in range(reps):
        nv.nvsm_profile_read(ctx)
        nv.nvsm_reconstruct_batch(ctx, p, bursts, ws)
        torch.cuda.synchronize()
        best = min(best, nv.nvsm_profile_read(ctx)["synthesize"][0])
    together = [b[2].clone() for b in bursts]
    for (fr, s, out), ref in zip(bursts, together):
        out.fill_(float("nan"))
        nv.nvsm_reconstruct(ctx, p, fr, s, out, ws)
        assert torch.equal(out, ref) and torch.isfinite(out).all()
    nv.nvsm_destroy(ctx)
    return best


@pytest.mark.parametrize("shapes,stride", [
    ([(2, 64, 64), (1, 64, 2000), (2, 700, 64), (1, 100, 1028)], 32),        # four pixels per thread
    ([(2, 65, 64), (1, 64, 2001), (2, 700, 65), (1, 100, 1030)], 32),        # one
    ([(1, 64, 64), (1, 80, 72)], 30)])
def test_images_of_a_batch_are_those_alone(shapes, stride):
    _run(shapes, stride)


def test_one_wide_image_among_tall_ones_costs_its_pixels():
    """Sixteen tall images, and fifteen with a wide one of the same pixels: the
    same work (twenty times slower where every row took the widest's width)."""
    from gpu_helpers import say
    tall = _run([(1, 16384, 64)] * 16, 64, 4)
    mixed = _run([(1, 64, 16384)] + [(1, 16384, 64)] * 15, 64, 4)
    say(f"synthesis of 16 tall images {tall:.3f} ms, one of them wide {mixed:.3f} ms")
    assert mixed <= 2 * tall
