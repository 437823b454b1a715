"""GPU checks of maps that nearly all rays meet in a few pixels, where a row's, a wave's or a workgroup's rays are added
at once: one pixel, pixels whose edges cross the rows and columns, maps beside which some or all rays fall, ragged
windows.  The counts must be those of the rays' own pixels, singly and in a batch; an explicit map window, which
these kernels do not take, changes nothing.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_lens", [0, 16, 100, 300, 2100])
@pytest.mark.parametrize("win", [((0, 0), (1024, 512)), ((3, 2), (70, 9)), ((1, 1), (10, 3000)), ((0, 5), (300, 1))])
def test_counts_are_those_of_the_rays(n_lens, win):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    print(f"few pixels: {n_lens} lenses, window {win}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(n_lens + win[1][0])
    lenses = torch.rand((n_lens, 4), device=dev, generator=g)
    lenses[:, :2] = 30.0 * lenses[:, :2] - 15.0
    rays = win[1][0] * win[1][1]
    y = torch.empty((rays, 2), dtype=torch.float64, device=dev)
    pix = torch.empty(rays, dtype=torch.int32, device=dev)
    jobs, maps, wants = [], [], []
    for lo, hi, n in (((-1e4, -1e4), (1e4, 1e4), (1, 1)), ((-900.0, -0.01), (900.0, 900.0), (1, 2)), ((-0.3, -500.0), (400.0, 500.0), (3, 1)),
                      ((-60.0, -60.0), (60.0, 60.0), (4, 4)), ((900.0, 900.0), (901.0, 901.0), (2, 2))):
        for window in (0, 64):
            o = P.Opts()
            o.block_cols, o.block_rows, o.map_window = 1, 4, window
            o.ray_y, o.ray_pix = y.data_ptr(), pix.data_ptr()
            counts = torch.zeros((n[1], n[0]), dtype=torch.int32, device=dev)
            lost = torch.zeros(1, dtype=torch.int64, device=dev)
            args = (lenses, 0.1, 0.2, (-12.0, -11.0), (12.0, 13.0), (1100, 3100), lo, hi, n)
            job = P.make_job(*args, counts, lost, window=win)
            P.shoot_job(job, torch.empty(P.workspace_bytes(job, o), dtype=torch.uint8, device=dev), o)
            want = torch.bincount(pix[pix >= 0].long(), minlength=n[0] * n[1]).cpu()
            assert torch.equal(counts.view(-1).cpu().long(), want), (n, window)
            assert int(lost.item()) == int((pix < 0).sum()) == rays - int(want.sum()), (n, window)
        wants.append((want, int(lost.item())))
        maps.append((torch.zeros((n[1], n[0]), dtype=torch.int32, device=dev), torch.zeros(1, dtype=torch.int64, device=dev)))
        jobs.append(P.make_job(*args, *maps[-1], window=win))
    P.shoot_batched(jobs, torch.empty(P.batched_workspace_bytes(jobs), dtype=torch.uint8, device=dev))
    for k, ((counts, lost), (want, want_lost)) in enumerate(zip(maps, wants)):
        assert torch.equal(counts.view(-1).cpu().long(), want) and int(lost.item()) == want_lost, k
