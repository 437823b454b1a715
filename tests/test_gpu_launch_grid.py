"""GPU checks of launches of 2^32 threads or more: a ray window one column wide, whole against in parts, through
each kernel of the one-column blocks (eight waves a workgroup, four, and the unsplit one).
"""
import pytest

pytestmark = pytest.mark.gpu


def _env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0905_2453_amd as P
    P.lib()
    return torch, P


@pytest.mark.parametrize("n_lens,rows", [(2048, (1 << 25) + 701), (65, (1 << 26) + 1000), (3, (1 << 28) + 5000)])
def test_strip_equals_its_parts(n_lens, rows):
    torch, P = _env()
    print(f"strip of {rows} rays, {n_lens} lenses", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n_lens)
    lenses = torch.rand((n_lens, 4), device="cuda", generator=g)
    lenses[:, :2] = 40.0 * lenses[:, :2] - 20.0
    half, out = 3 << 23, []
    for parts in ([(0, rows)], [(0, half), (half, rows - half)] if rows < 2 * half
                  else [(b, min(half, rows - b)) for b in range(0, rows, half)]):
        counts = torch.zeros((64, 64), dtype=torch.int32, device="cuda")
        lost = torch.zeros(1, dtype=torch.int64, device="cuda")
        for b, n in parts:
            P.shoot(lenses, 0.1, 0.2, (-16.0, -16.0), (16.0, 16.0), (64, rows), (-8.0, -8.0), (8.0, 8.0), (64, 64),
                    counts=counts, lost=lost, window=((40, b), (1, n)))
        out.append((counts.cpu(), int(lost.item())))
    assert int(out[0][0].sum()) + out[0][1] == rows
    assert torch.equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]
