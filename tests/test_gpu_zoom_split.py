"""GPU checks of the culling kernel's split of the lenses over waves and lanes: lens counts around the
chunks of 64 that a wave takes and the sixteen waves of a workgroup, cell counts that leave its last
workgroup part empty, one to a few cells, and moving lenses.  The zoom must add exactly the counts of
the plain shoot of the same job, and shoot no more than all of its rays.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_lens,rays,cell,moving", [
    (1, (40, 36), (5, 4), False),
    (63, (301, 211), (0, 0), False),
    (64, (64, 64), (64, 64), False),
    (65, (517, 130), (3, 8), True),
    (1023, (400, 400), (8, 8), False),
    (1025, (1200, 900), (0, 0), False),
    (2100, (2000, 64), (1, 4), True),
])
def test_zoom_counts_equal_plain(n_lens, rays, cell, moving):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    print(f"zoom culling: {n_lens} lenses, {rays} rays, cells {cell}", flush=True)
    dev = torch.device("cuda:0")
    lenses_np, r = synth.lens_field(80 + n_lens, n_lens, kappa_star=0.4)
    lenses = torch.from_numpy(lenses_np).to(dev)
    vel = torch.from_numpy(synth.lens_velocities(3, n_lens, 0.2)).to(dev) if moving else None
    half = (0.5 * r + 1.0, 0.4 * r + 1.0)
    out = []
    for zoom in (False, True):
        counts = torch.zeros((40, 50), dtype=torch.int32, device=dev)
        lost = torch.zeros(1, dtype=torch.int64, device=dev)
        job = P.make_job(lenses, 0.0, 0.15, (-half[0], -half[1]), half, rays, (-0.3 * half[0], -0.1), (0.2, 0.3 * half[1]),
                         (50, 40), counts, lost, velocities=vel, time=0.7)
        if zoom:
            z = P.zoom_params(cell)
            ws = torch.empty(P.zoom_workspace_bytes(job, z), dtype=torch.uint8, device=dev)
            P.shoot_zoom(job, z, ws)
            st = P.zoom_stats(ws)
            assert st["cells_kept"] <= st["cells"] and st["slots_shot"] <= st["slots"]
        else:
            P.shoot_job(job, torch.empty(P.workspace_bytes(job), dtype=torch.uint8, device=dev))
        torch.cuda.synchronize()
        out.append(counts.cpu().numpy().view(np.uint32))
    assert out[0].sum() > 0
    assert np.array_equal(out[0], out[1])
