"""Frame statistics of a burst of few patches, whose frame pairs spread over
the card, against the same patches within a burst of many, where a workgroup
walks its frame group: the sums are the same operations in the same order."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,F,dtype", [(64, 1, "float32"), (64, 20, "uint16"), (64, 21, "float32"),
                                       (64, 59, "uint16"), (128, 2, "uint16"), (128, 41, "float32")])
def test_few_patches_equal_the_same_among_many(N, F, dtype):
    import torch
    import paper_1701_00581_amd as nv
    p = nv.default_params(N, v_radius=3)
    big, small = 12, 2                         # patches per side: above and below the dividing line
    L, S = N + (big - 1) * N // 2, N + (small - 1) * N // 2
    g = torch.Generator(device="cuda").manual_seed(F)
    frames = (torch.rand(F, L, L, device="cuda", generator=g) * 3000).to(getattr(torch, dtype))
    many, few = nv.Session(p, L, L, F), nv.Session(p, S, S, F)
    many.accumulate(frames)
    few.accumulate(frames[:, :S, :S].contiguous())
    torch.cuda.synchronize()
    rows = [y * big + x for y in range(small) for x in range(small)]
    for a, b in ((many.power, few.power), (many.mean_spec, few.mean_spec), (many.mu, few.mu),
                 (many.bispec, few.bispec)):
        assert torch.equal(a[rows], b)
        assert torch.isfinite(torch.view_as_real(b) if b.is_complex() else b).all()
