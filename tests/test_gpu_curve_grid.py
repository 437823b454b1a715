"""GPU check of light curves of more than 2^24 points with a workgroup a point (2^32 threads or more), against the
same points one lane each.
"""
import pytest

pytestmark = pytest.mark.gpu


def _env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    return torch, P


def test_more_points_than_one_grid_dimension():
    torch, P = _env()
    g = torch.Generator(device="cuda").manual_seed(1)
    tracks, points = 4096, 4097                        # 2^24 + 4096 points
    counts = torch.randint(0, 100, (4, 4096), dtype=torch.int32, device="cuda", generator=g)
    ends = torch.rand((tracks, 4), dtype=torch.float64, device="cuda", generator=g) * 2.0 - 1.0
    # a box 260 columns wide and the map's four rows high, wider than a wave's staging area
    args = (counts, (-1.0, -0.001), (1.0, 0.001), (4096, 4), 3.0, ends * torch.tensor([0.9, 0.001, 0.9, 0.001],
            dtype=torch.float64, device="cuda"), points, "disc", 0.063)
    mu = [P.light_curve(*args, layout=k)[0] for k in ("waves", "lanes")]
    assert torch.equal(mu[0], mu[1])                   # a disc's sums are whole numbers
    assert bool(torch.isfinite(mu[0]).all())
