"""GPU checks of the zoom's blocks, counted through each row of cells by groups of four ray rows: rows of fewer
than 32 kept columns and of more, cells of one to many groups and of one to 64 columns, cells that start off a
multiple of four rows, more than 1024 cells to a row and rows of cells, windows, random ray positions.  The zoom
must add exactly the counts of the plain shoot of the same job.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_lens,rays,cell,window,jitter", [
    (40, (2600, 40), (1, 4), None, False), (300, (36, 4300), (9, 4), None, False), (3, (700, 500), (31, 13), None, False),
    (2100, (513, 400), (33, 5), ((5, 3), (500, 390)), False), (150, (640, 900), (64, 100), ((0, 1), (640, 897)), False),
    (500, (800, 800), (3, 24), None, False), (70, (900, 700), (2, 1), ((1, 2), (640, 511)), False),
    (260, (600, 700), (11, 6), ((7, 6), (300, 650)), True), (2049, (300, 300), (0, 0), None, True),
])
def test_row_blocks_equal_plain(n_lens, rays, cell, window, jitter):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    print(f"zoom rows: {n_lens} lenses, {rays} rays, cells {cell}, window {window}, jitter {jitter}", flush=True)
    dev = torch.device("cuda:0")
    lenses_np, r = synth.lens_field(30 + n_lens, n_lens, kappa_star=0.4)
    lenses = torch.from_numpy(lenses_np).to(dev)
    half = (0.5 * r + 1.0, 0.4 * r + 1.0)
    out = []
    for zoom in (False, True):
        counts = torch.zeros((40, 50), dtype=torch.int32, device=dev)
        lost = torch.zeros(1, dtype=torch.int64, device=dev)
        job = P.make_job(lenses, 0.0, 0.15, (-half[0], -half[1]), half, rays, (-0.3 * half[0], -0.1), (0.2, 0.3 * half[1]),
                         (50, 40), counts, lost, window=window, jitter_seed=9 if jitter else None)
        if zoom:
            z = P.zoom_params(cell)
            ws = torch.full((P.zoom_workspace_bytes(job, z),), 255, dtype=torch.uint8, device=dev)
            for again in range(2):               # a workspace as it comes, and as the last zoom left it
                counts.zero_()
                P.shoot_zoom(job, z, ws)
                st = P.zoom_stats(ws)
                assert 0 < st["cells_kept"] <= st["cells"] and st["slots_shot"] <= st["slots"]
                torch.cuda.synchronize()
                out.append(counts.cpu().numpy().view(np.uint32))
        else:
            P.shoot_job(job, torch.empty(P.workspace_bytes(job), dtype=torch.uint8, device=dev))
            torch.cuda.synchronize()
            out.append(counts.cpu().numpy().view(np.uint32))
    assert out[0].sum() > 0
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
