"""GPU checks of the choice between the one-column kernels at its limits: lens counts of two, three and eight groups
and a run more, windows of 2032 and 2048, 16368 and 16384 blocks, every run length, random positions.  Source positions are those of
the same rays shot as part of a small window (which another kernel takes), bit for bit: float32 group sums meet in
FP64, where they are exact.
"""
import pytest

pytestmark = pytest.mark.gpu

CASES = [(n, rows, 0, None) for n in (64, 65, 96, 97, 104, 105, 256, 257) for rows in (508, 511, 4092, 4096)]
CASES += [(n, rows, 16, None) for n in (128, 129, 300) for rows in (4092, 4096)]
CASES += [(n, rows, 32, None) for n in (31, 33, 129, 256, 257, 1025, 1100) for rows in (700, 4092, 4096)]
# random positions: four groups at 6144 blocks, 1023 lenses at 16384, eight waves from 4096 lenses on
CASES += [(n, rows, 0, 11) for n in (65, 128, 129) for rows in (1532, 1536)]
CASES += [(n, rows, 0, 12) for n in (600, 1023, 1024) for rows in (4092, 4096)] + [(n, 600, 0, 13) for n in (4095, 4096)]


@pytest.mark.parametrize("n_lens,rows,run,jitter", CASES)
def test_rays_do_not_depend_on_the_window(n_lens, rows, run, jitter):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    print(f"routes: {n_lens} lenses, {rows} rows, runs of {run}, jitter {jitter}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(n_lens)
    lenses = torch.rand((n_lens, 4), device=dev, generator=g)
    lenses[:, :2] = 30.0 * lenses[:, :2] - 15.0
    cols = 500 if rows == 700 else 1024
    y = {}
    for name, win in (("whole", ((0, 0), (cols, rows))), ("part", ((cols - 70, rows - 41), (70, 41)))):
        n = win[1][0] * win[1][1]
        o = P.Opts()
        o.fp32_run = run
        yy = torch.empty((n, 2), dtype=torch.float64, device=dev)
        pix = torch.empty(n, dtype=torch.int32, device=dev)
        o.ray_y, o.ray_pix = yy.data_ptr(), pix.data_ptr()
        counts, lost = P.shoot(lenses, 0.1, 0.2, (-12.0, -11.0), (12.0, 13.0), (cols, rows), (-6.0, -6.0), (6.0, 6.0),
                               (64, 50), window=win, opts=o, jitter_seed=jitter)
        assert torch.equal(counts.view(-1).cpu(), torch.bincount(pix[pix >= 0].long(), minlength=3200).int().cpu())
        assert int(counts.sum()) + int(lost.item()) == n
        y[name] = yy.view(win[1][1], win[1][0], 2)
    assert torch.equal(y["whole"][-41:, -70:].contiguous().view(torch.int64), y["part"].contiguous().view(torch.int64))
