"""GPU checks of the light curves' wave layouts: one wave per point, with and without pixels requested ahead, and
one workgroup per point, with its support box staged and beyond the staging area.  Cases run from one point to
thousands, boxes from one pixel over the last few of a request to more than a workgroup's staging, cut by
the map's edges.  Disc sums are sums of integers and must equal the oracle's bit for bit; Gaussian sums of up to
1e6 positive terms, at most 4e3 of them in one chain, differ by less than 1e-12.
"""
import numpy as np
import pytest

import synth
from oracle import lightcurve as lc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,size,n,tracks,points", [
    ("disc", 1.3, (40, 31), 1, 1), ("disc", 1.9, (64, 64), 3, 17), ("disc", 2.05, (301, 77), 5, 60),      # workgroups
    ("disc", 20.0, (333, 290), 2, 9), ("gaussian", 6.0, (420, 530), 1, 13),                              # boxes over 128
    ("disc", 70.0, (1300, 41), 1, 11), ("gaussian", 18.0, (1220, 90), 2, 5),                               # boxes over 512
    ("disc", 3.6, (90, 120), 9, 170), ("gaussian", 0.9, (90, 120), 5, 301),                              # ahead
    ("disc", 0.4, (50, 40), 40, 211), ("gaussian", 0.2, (50, 41), 67, 90),                               # one by one
])
def test_wave_layouts_match_oracle(kind, size, n, tracks, points):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    print(f"light-curve waves: {kind} {size} {n} {tracks} x {points}", flush=True)
    lo = (-2.0, 1.0)
    hi = (lo[0] + 0.25 * n[0], lo[1] + 0.25 * n[1])
    counts = synth.count_map(5, n, 40.0)
    tr = np.array(synth.light_tracks(6, tracks, lo, hi, 3.0))
    dev = torch.device("cuda:0")
    c = torch.from_numpy(counts.view(np.int32).copy()).to(dev)
    mu, _ = P.light_curve(c, lo, hi, n, 25.0, torch.from_numpy(tr).to(dev), points, kind, size, layout=2)
    torch.cuda.synchronize()
    mu = mu.cpu().numpy()
    mu_o, _ = lc.light_curve(counts, lo, hi, n, 25.0, tr, points, kind, size)
    assert np.array_equal(np.isnan(mu), np.isnan(mu_o)) and (~np.isnan(mu_o)).any()
    ok = ~np.isnan(mu_o)
    if kind == "disc":
        assert np.array_equal(mu[ok], mu_o[ok])
    else:
        assert np.all(np.abs(mu[ok] - mu_o[ok]) <= 1e-12 * np.abs(mu_o[ok]))
