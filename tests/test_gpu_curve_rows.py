"""GPU checks of the light curves' lane layout at the ends of a row's run of pixels: runs of zero to a few
pixels (every remainder of the four-wide loads), runs cut by each edge of the map, pixel centres exactly on
the support's edge, sources off the map, and maps far from the origin, where rounding moves the pixels'
places.  Disc sums are sums of integers and must equal the oracle's bit for bit; Gaussian ones agree to 1e-12.
"""
import numpy as np
import pytest

import synth
from oracle import lightcurve as lc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,size,lo,n", [
    ("disc", 0.26, (0.0, 0.0), (40, 31)), ("disc", 1.0, (-3.0, 2.0), (40, 31)), ("disc", 1.625, (0.0, 0.0), (41, 33)),
    ("disc", 0.9, (1.0e6, -2.0e6), (37, 29)), ("disc", 30.0, (0.0, 0.0), (19, 5)), ("disc", 0.5, (4096.0, 0.0), (3, 200)),
    ("gaussian", 0.11, (0.0, 0.0), (40, 31)), ("gaussian", 0.4, (-2.0, -1.0), (39, 30)), ("gaussian", 0.3, (1.0e5, 7.0), (64, 9)),
])
def test_lane_rows_match_oracle(kind, size, lo, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    print(f"light-curve rows: {kind} {size} {lo} {n}", flush=True)
    hi = (lo[0] + 0.25 * n[0], lo[1] + 0.25 * n[1])          # pixels of 1/4: centres and radii meet exactly
    counts = synth.count_map(9, n, 40.0)
    on = [[lo[0] + 1.125, lo[1] + 1.125, hi[0] - 1.125, lo[1] + 1.125],       # centre to centre along a row
          [lo[0] + 2.0, lo[1] - 1.0, lo[0] + 2.0, hi[1] + 1.0],               # down a pixel edge, off both ends
          [lo[0] - 1.0, lo[1] + 0.3, hi[0] + 1.0, hi[1] - 0.3], [hi[0], hi[1], lo[0], lo[1]],
          [lo[0] + 0.125, lo[1] + 0.125, lo[0] + 0.126, lo[1] + 0.125]]
    tr = np.concatenate([np.array(on), synth.light_tracks(4, 12, lo, hi, 3.0)])
    dev = torch.device("cuda:0")
    c = torch.from_numpy(counts.view(np.int32).copy()).to(dev)
    mu, mag = P.light_curve(c, lo, hi, n, 25.0, torch.from_numpy(tr).to(dev), 57, kind, size, layout=1)
    torch.cuda.synchronize()
    mu, mag = mu.cpu().numpy(), mag.cpu().numpy()
    mu_o, mag_o = lc.light_curve(counts, lo, hi, n, 25.0, tr, 57, kind, size)
    assert np.array_equal(np.isnan(mu), np.isnan(mu_o)) and (~np.isnan(mu_o)).any()
    ok = ~np.isnan(mu_o)
    if kind == "disc":
        assert np.array_equal(mu[ok], mu_o[ok])
    else:
        assert np.all(np.abs(mu[ok] - mu_o[ok]) <= 1e-12 * np.abs(mu_o[ok]))
