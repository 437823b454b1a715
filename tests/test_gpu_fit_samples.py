"""GPU checks of the exact far-field samples at the edges of their launches: lens counts around the groups
of 64 that a wave takes and the waves of a workgroup, and fits on both sides of each choice of kernel and
waves per workgroup (256, 16384 and 32768 blocks of 256 samples).

Every residual sample of a few tiles against the FP64 oracle within the float32 forward-error bound
(8 + 16 + 4) 2^-24 sum m / r plus the float32 rounding of the stored residual; and the tiles that a
small and a large fit share must have the same targets bit for bit.
"""
import numpy as np
import pytest

import synth
from oracle import farfield as off

pytestmark = pytest.mark.gpu


def _targets(n_lens, tiles, n_samples, shared, tile=(8, 8), r_near=1.5, kappa=0.5):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    dev = torch.device("cuda:0")
    lenses, r = synth.lens_field(30 + n_lens, n_lens, kappa_star=kappa)
    n = (2048, 2048)
    w = synth.Workload("samples", lenses, 0.0, 0.0, (-40.0, -30.0), (40.0, 30.0), n, (-3.0, -3.0), (3.0, 3.0), (16, 16))
    win = ((1000, 1003), (tiles[0] * tile[0], tiles[1] * tile[1]))
    u = synth.fit_samples_quads(5, n_samples) if shared else synth.fit_samples(5, n_samples)
    nt = tiles[0] * tiles[1]
    counts = torch.zeros((16, 16), dtype=torch.int32, device=dev)
    lost = torch.zeros(1, dtype=torch.int64, device=dev)
    job = P.make_job(torch.from_numpy(lenses).to(dev), 0.0, 0.0, w.grid_lo, w.grid_hi, n, w.map_lo, w.map_hi, w.map_n, counts,
                     lost, window=win)
    dt = torch.full((nt, n_samples, 2), float("nan"), dtype=torch.float32, device=dev)
    cfg = P.ff_config(torch.from_numpy(u).to(dev), torch.from_numpy(synth.init_params(5)).to(dev), tile_rays=tile,
                      r_near=r_near, steps=0, batch=256, debug_targets=dt, shared_x=shared)
    u8 = dict(dtype=torch.uint8, device=dev)
    P.farfield_fit(job, cfg, torch.empty(P.farfield_model_bytes(job, cfg), **u8),
                   torch.empty(P.farfield_fit_workspace_bytes(job, cfg), **u8))
    torch.cuda.synchronize()
    return w, win, u, dt.cpu().numpy()


@pytest.mark.parametrize("n_lens,tiles,n_samples,shared", [
    (1, (2, 1), 1024, True), (63, (3, 1), 1024, False), (64, (1, 1), 2048, True), (65, (2, 2), 1024, False),
    (1025, (8, 8), 1024, True),       # 256 blocks: sixteen waves
    (1025, (13, 5), 1024, True),      # 260: eight
    (511, (64, 65), 1024, False),     # 16640: four
])
def test_samples_against_oracle(n_lens, tiles, n_samples, shared):
    print(f"far-field samples: {n_lens} lenses, {tiles} tiles of {n_samples}", flush=True)
    w, win, u, got = _targets(n_lens, tiles, n_samples, shared)
    assert np.isfinite(got).all()
    worst = 0.0
    for t in sorted({0, len(got) // 2, len(got) - 1}):
        res, _, _, _, far = off.tile_targets(w, win, (8, 8), t % tiles[0], t // tiles[0], 1.5, u)
        _, _, c, h, _ = off.tile_rect(w, win, (8, 8), t % tiles[0], t // tiles[0])
        p = (c + u.astype(np.float64) * h).astype(np.float32).astype(np.float64)
        L = w.lenses[far].astype(np.float64)
        s = np.sum(L[None, :, 2] / np.hypot(p[:, None, 0] - L[None, :, 0], p[:, None, 1] - L[None, :, 1]), 1)
        bound = (8 + 16 + 4) * 2.0 ** -24 * s[:, None] + 2.0 ** -23 * np.abs(res) + 1e-12
        worst = max(worst, float((np.abs(got[t] - res) / bound).max()))
    print(f"  worst error {worst:.3f} of the bound", flush=True)
    assert worst <= 1.0


def test_small_and_large_fits_share_targets():
    # 8192 tiles of 1024 samples (the kernel for large fits) against the first row of tiles alone
    big = _targets(777, (128, 64), 1024, True)[3]
    small = _targets(777, (128, 1), 1024, True)[3]
    assert np.isfinite(big).all() and np.array_equal(big[:128], small)
