"""GPU checks of the closure's evaluation kernel and of the moving field's affine bases at the edges of their
launches: tiles narrower than a wave and rows that do not come in fours, tiles shared by many workgroups,
candidate lists that fill less than a run, several runs and several batches of the LDS stage, random ray
positions, and affine bases summed by 1, some and 64 workgroups per tile.

With the network off, every ray's source position against the FP64 oracle: the exact affine base at the
tile centre plus the near lenses, within the near sum's float32 forward-error bound
(8 + 16) 2^-24 sum m / r plus 1e-10 of the affine part.  The dumped pixels must make up the map.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

# lenses, rays, tile, r_near, jitter seed, moving
CASES = [
    (300, (37, 23), (5, 3), 2.0, None, False),
    (300, (64, 64), (64, 64), 3.0, 4, False),
    (2000, (130, 101), (64, 50), 1.0, None, True),      # lists of a few runs, most of their lenses far
    (2000, (200, 70), (100, 70), 5.0, 11, True),
    (6000, (96, 66), (96, 66), 40.0, None, False),      # one tile whose candidates fill several batches
    (6000, (96, 66), (32, 33), 40.0, 3, True),
    (17, (300, 9), (300, 9), 0.5, None, True),          # fewer lenses than a workgroup's threads
    (30000, (70, 70), (1, 70), 1.5, None, True),        # columns of one ray
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"n{c[0]}-{c[1][0]}x{c[1][1]}-tile{c[2][0]}x{c[2][1]}")
def test_affine_and_near_field_per_ray(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    n, rays, tile, r_near, jseed, moving = case
    print(f"closure evaluation: {case}", flush=True)
    dev = torch.device("cuda:0")
    lenses, r = synth.lens_field(20 + n, n, kappa_star=0.5)
    lo, hi = (-0.2 * min(r, 20.0), -0.15 * min(r, 20.0)), (0.2 * min(r, 20.0), 0.2 * min(r, 20.0))
    counts = torch.zeros((33, 45), dtype=torch.int32, device=dev)
    lost = torch.zeros(1, dtype=torch.int64, device=dev)
    mlo, mhi = (-2.0, -1.5), (2.0, 1.5)
    lt = torch.from_numpy(lenses).to(dev)
    args = (lt, 0.05, 0.1, lo, hi, rays, mlo, mhi, (45, 33), counts, lost)
    job = P.make_job(*args, jitter_seed=jseed)
    cfg = P.ff_config(torch.from_numpy(synth.fit_samples(7, 1024)).to(dev), torch.from_numpy(synth.init_params(7)).to(dev),
                      tile_rays=tile, r_near=r_near, steps=0, batch=256)
    u8 = dict(dtype=torch.uint8, device=dev)
    model = torch.empty(P.farfield_model_bytes(job, cfg), **u8)
    P.farfield_fit(job, cfg, model, torch.empty(P.farfield_fit_workspace_bytes(job, cfg), **u8))
    vel = synth.lens_velocities(5, n, 0.1)
    shot = P.make_job(*args, jitter_seed=jseed, velocities=torch.from_numpy(vel).to(dev), time=0.8) if moving else job
    nr = rays[0] * rays[1]
    ry = torch.full((nr, 2), float("nan"), dtype=torch.float64, device=dev)
    rp = torch.full((nr,), -7, dtype=torch.int32, device=dev)
    o = P.Opts()
    o.ray_y, o.ray_pix, o.flags = ry.data_ptr(), rp.data_ptr(), P._abi.RS_FLAG_AFFINE_ONLY
    P.farfield_eval(shot, cfg, model, torch.empty(P.farfield_eval_workspace_bytes(shot, cfg), **u8), o)
    torch.cuda.synchronize()
    y, pix = ry.cpu().numpy(), rp.cpu().numpy()
    c = counts.cpu().numpy().view(np.uint32).ravel()
    assert pix.min() >= -1
    assert np.array_equal(c, np.bincount(pix[pix >= 0], minlength=c.size)) and int(lost.item()) == int(np.sum(pix == -1))
    # the same split in FP64: near and far by the fit-time positions, sums at the moved ones
    at = (oracle.lenses_at(lenses, vel, 0.8) if moving else lenses).astype(np.float64)
    fit = lenses.astype(np.float64)
    t = [(hi[k] - lo[k]) / rays[k] for k in range(2)]
    u = [np.full((rays[1], rays[0]), 0.5)] * 2
    if jseed is not None:
        idx = np.arange(nr, dtype=np.uint64)
        key = [synth.stream_key(jseed, 8 + k) for k in range(2)]
        with np.errstate(over="ignore"):
            u = [((synth.mix64(key[k] + (idx + np.uint64(1)) * synth.GOLDEN) >> np.uint64(11)).astype(np.float64) * 2.0 ** -53)
                 .reshape(rays[1], rays[0]) for k in range(2)]
    lam = ((1.0 - 0.1) - 0.05, (1.0 + 0.1) - 0.05)
    worst = 0.0
    for ty in range(0, rays[1], tile[1]):
        for tx in range(0, rays[0], tile[0]):
            e = (min(tx + tile[0], rays[0]), min(ty + tile[1], rays[1]))
            a, b = np.array([lo[0] + tx * t[0], lo[1] + ty * t[1]]), np.array([lo[0] + e[0] * t[0], lo[1] + e[1] * t[1]])
            gap = np.maximum(np.maximum(a - fit[:, :2], fit[:, :2] - b), 0.0)
            near = (gap * gap).sum(1) < r_near * r_near
            cen = 0.5 * (a + b)
            d, m = cen - at[~near, :2], at[~near, 2]
            r2 = (d * d).sum(1)
            a0 = (m[:, None] * d / r2[:, None]).sum(0)
            j11, j12 = (m * (d[:, 1] ** 2 - d[:, 0] ** 2) / r2 ** 2).sum(), (-2.0 * m * d[:, 0] * d[:, 1] / r2 ** 2).sum()
            i1, i2 = np.meshgrid(np.arange(tx, e[0]), np.arange(ty, e[1]))
            x = [(lo[0] + (i1 + u[0][i2, i1]) * t[0]).astype(np.float32).astype(np.float64).ravel(),
                 (lo[1] + (i2 + u[1][i2, i1]) * t[1]).astype(np.float32).astype(np.float64).ravel()]
            f = [a0[0] + j11 * (x[0] - cen[0]) + j12 * (x[1] - cen[1]), a0[1] + j12 * (x[0] - cen[0]) - j11 * (x[1] - cen[1])]
            s = np.zeros(len(x[0]))
            for q in at[near]:
                dx, dy = x[0] - q[0], x[1] - q[1]
                q2 = dx * dx + dy * dy
                f[0], f[1] = f[0] + q[2] * dx / q2, f[1] + q[2] * dy / q2
                s += q[2] / np.sqrt(q2)
            got = y[(i2 * rays[0] + i1).ravel()]
            want = np.stack([lam[0] * x[0] - f[0], lam[1] * x[1] - f[1]], 1)
            bound = (8 + 16) * 2.0 ** -24 * s + 1e-10 * (1.0 + np.abs(a0).sum())
            worst = max(worst, float((np.abs(got - want).max(1) / bound).max()))
    print(f"  worst error {worst:.3f} of the bound", flush=True)
    assert worst <= 1.0
