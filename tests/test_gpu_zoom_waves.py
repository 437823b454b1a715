"""GPU checks of the zoom at its choices by lens count: the waves of a culling workgroup (lens counts around each
multiple of 64 at which they change, and around the eight chunks of the largest), lanes per cell by the cells that
are left, the two shooting kernels, run lengths, random ray positions and moving lenses.  The zoom must add exactly
the counts of the plain shoot of the same job.
"""
import pytest

pytestmark = pytest.mark.gpu

CASES = [(n, 1.0, 0, None, False) for n in (0, 2, 64, 65, 128, 129, 256, 257, 383, 384, 511, 512, 513)]
CASES += [(n, 0.05, 0, None, False) for n in (1, 64, 100, 200, 256)]          # few cells left: four lanes each
CASES += [(n, 20.0, 0, None, False) for n in (64, 127, 192)]                  # all cells kept: a lane each
CASES += [(40, 1.0, 16, 7, False), (130, 2.0, 32, 9, True), (250, 2.0, 0, 3, True), (383, 1.0, 32, None, True), (600, 1.0, 32, 5, False)]


@pytest.mark.parametrize("n_lens,side,run,jitter,moving", CASES)
def test_zoom_counts_equal_plain(n_lens, side, run, jitter, moving):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    print(f"zoom: {n_lens} lenses, side {side}, runs of {run}, jitter {jitter}, moving {moving}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(n_lens + 1)
    lenses = torch.rand((n_lens, 4), device=dev, generator=g)
    lenses[:, :2] = 30.0 * lenses[:, :2] - 15.0
    vel = 0.2 * torch.randn((n_lens, 2), device=dev, generator=g) if moving else None
    o = P.Opts()
    o.fp32_run = run
    out = []
    for zoom in (False, True):
        counts = torch.zeros((40, 50), dtype=torch.int32, device=dev)
        lost = torch.zeros(1, dtype=torch.int64, device=dev)
        job = P.make_job(lenses, 0.0, 0.15, (-20.0, -19.0), (20.0, 21.0), (2000, 1901), (0.5 - side / 2, -side / 2),
                         (0.5 + side / 2, side / 2), (50, 40), counts, lost, window=((3, 2), (1990, 1891)),
                         jitter_seed=jitter, velocities=vel, time=0.7)
        if zoom:
            z = P.zoom_params()
            ws = torch.empty(P.zoom_workspace_bytes(job, z, o), dtype=torch.uint8, device=dev)
            P.shoot_zoom(job, z, ws, o)
            st = P.zoom_stats(ws)
            assert st["cells_kept"] <= st["cells"] and st["slots_shot"] <= st["slots"]
        else:
            P.shoot_job(job, torch.empty(P.workspace_bytes(job, o), dtype=torch.uint8, device=dev), o)
        out.append(counts.cpu())
    assert int(out[0].sum()) > 0
    assert torch.equal(out[0], out[1])
