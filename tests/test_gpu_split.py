"""GPU checks of the one-column kernels that split the lenses over a workgroup's waves (k_split), at the
edges of their dispatch: lens counts around the groups of 32, 64 and 128 lenses that a wave takes,
block counts on both sides of each choice of waves per workgroup, ragged windows, every float32 run
length, staged tile, random ray positions and moving lenses.

Every ray's source position against the FP64 oracle within the plain path's float32 forward-error
bound, (8 + 16) 2^-24 sum m / r; lost rays, map and per-ray pixels are checked exactly against each
other.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

# lenses, window start and size, float32 run, lens tile, jitter seed, moving
CASES = [
    (1, (0, 0), (70, 9), 0, 0, None, False),
    (33, (3, 2), (64, 4), 0, 0, None, False),
    (65, (1, 1), (130, 7), 0, 0, 5, False),
    (127, (0, 3), (61, 5), 0, 0, None, True),
    (128, (0, 0), (65, 17), 0, 0, None, False),
    (513, (7, 5), (200, 30), 0, 0, None, False),       # sixteen waves, one group past a full round
    (2049, (0, 0), (100, 50), 0, 0, 9, True),
    (300, (0, 1), (640, 300), 0, 0, None, False),      # eight waves: few blocks
    (255, (0, 1), (640, 300), 0, 0, None, False),      # four
    (2050, (2, 2), (700, 750), 0, 0, None, False),     # eight: a large field
    (100, (0, 0), (1200, 600), 0, 0, None, False),     # four: many blocks
    (64, (0, 0), (2100, 260), 0, 0, None, False),      # two groups: the row-tiled kernel ...
    (65, (0, 0), (2100, 260), 0, 0, None, False),      # ... and three
    (200, (5, 3), (90, 41), 16, 0, None, False),
    (1100, (0, 0), (90, 41), 16, 512, 2, False),
    (129, (5, 3), (90, 41), 32, 0, None, False),
    (1025, (0, 2), (300, 33), 8, 512, None, True),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"n{c[0]}-{c[2][0]}x{c[2][1]}-T{c[3]}-LT{c[4]}")
def test_split_rays_against_oracle(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    n, w0, wn, T, LT, jseed, moving = case
    print(f"split kernel: {case}", flush=True)
    dev = torch.device("cuda:0")
    grid = (w0[0] + wn[0] + 3, w0[1] + wn[1] + 2)
    lenses, r = synth.lens_field(50 + n, n, kappa_star=0.4)
    # the window lies in the middle third of the lens disc
    lo, hi = (-0.4 * r - 1.0, -0.3 * r - 1.0), (0.4 * r + 1.0, 0.3 * r + 1.1)
    vel = synth.lens_velocities(7, n, 0.3)
    at = oracle.lenses_at(lenses, vel, 1.25) if moving else lenses
    w = synth.Workload("split", at, 0.1, 0.2, lo, hi, grid, (-3.0, -2.0), (3.0, 2.5), (61, 47), jitter_seed=jseed)
    rays = wn[0] * wn[1]
    o = P.Opts()
    ry = torch.full((rays, 2), float("nan"), dtype=torch.float64, device=dev)
    rp = torch.full((rays,), -7, dtype=torch.int32, device=dev)
    o.ray_y, o.ray_pix, o.fp32_run, o.lens_tile = ry.data_ptr(), rp.data_ptr(), T, LT
    counts = torch.zeros((47, 61), dtype=torch.int32, device=dev)
    lost = torch.zeros(1, dtype=torch.int64, device=dev)
    job = P.make_job(torch.from_numpy(lenses).to(dev), 0.1, 0.2, lo, hi, grid, w.map_lo, w.map_hi, w.map_n, counts, lost,
                     window=(w0, wn), jitter_seed=jseed, velocities=torch.from_numpy(vel).to(dev) if moving else None,
                     time=1.25)
    P.shoot_job(job, torch.empty(P.workspace_bytes(job, o), dtype=torch.uint8, device=dev), o)
    torch.cuda.synchronize()
    y, pix = ry.cpu().numpy(), rp.cpu().numpy().astype(np.int64)
    c = counts.cpu().numpy().view(np.uint32).ravel()
    assert np.array_equal(c, np.bincount(pix[pix >= 0], minlength=c.size)) and int(lost.item()) == int(np.sum(pix == -1))
    assert pix.min() >= -1
    # a seeded part of the rays, and the window's corners and last row
    idx = np.unique(np.concatenate([synth.sample_indices(3, rays, 4000), np.arange(rays - wn[0], rays), [0, wn[0] - 1]]))
    i1, i2 = w0[0] + idx % wn[0], w0[1] + idx // wn[0]
    y_o, p_o = oracle.trace_parallel(w, i2 * grid[0] + i1)
    if jseed is None:
        x = np.stack([oracle.axis(lo[0], hi[0], grid[0]).astype(np.float64)[i1],
                      oracle.axis(lo[1], hi[1], grid[1]).astype(np.float64)[i2]], 1)
    else:                              # anywhere in the cell: the bound of the nearest corner holds up to the cell
        x = np.stack([lo[0] + (i1 + 0.5) * (hi[0] - lo[0]) / grid[0], lo[1] + (i2 + 0.5) * (hi[1] - lo[1]) / grid[1]], 1)
    L = at.astype(np.float64)
    d = np.hypot(x[:, 0, None] - L[None, :, 0], x[:, 1, None] - L[None, :, 1])
    if jseed is not None:
        half = 0.5 * np.hypot((hi[0] - lo[0]) / grid[0], (hi[1] - lo[1]) / grid[1])
        d = np.maximum(d - half, 1e-3)
    bound = (8 + 16) * 2.0 ** -24 * np.sum(L[None, :, 2] / d, 1) + 1e-12
    ok = np.isfinite(y_o).all(1)
    err = np.abs(y[idx] - y_o).max(1)
    assert np.all(err[ok] <= bound[ok]), float((err[ok] / bound[ok]).max())
    # pixels differ only where the oracle's position lies within the bound of a pixel edge
    px = [(w.map_hi[k] - w.map_lo[k]) / w.map_n[k] for k in range(2)]
    f = [(y_o[:, k] - w.map_lo[k]) / px[k] for k in range(2)]
    with np.errstate(invalid="ignore"):
        edge = np.minimum(*[np.abs(f[k] - np.round(f[k])) * px[k] for k in range(2)])
        assert np.all((pix[idx] == p_o) | ~(edge > bound))
