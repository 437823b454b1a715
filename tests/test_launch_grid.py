"""Launch shapes of very many workgroups (no GPU): csrc/launch_grid.h, compiled as the library includes it."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0905_2453_amd", "csrc")


def _blocks(n1, n2, rows=4):
    return -(-n1 // 64) * -(-n2 // rows)


@pytest.mark.parametrize("n,threads", [
    (1, 256), (257, 1024), (8388607, 512), (8388608, 512),
    (_blocks(46340, 46340), 512), (_blocks(32768, 65535), 512), (_blocks(10, 33600000), 512), (_blocks(46340, 46340), 256),
    (_blocks(1, 2 ** 31 - 1), 512), (_blocks(1, 2 ** 31 - 1), 256), (_blocks(1, 2 ** 31 - 1, 16), 256), (2 ** 24, 256),
    (2 ** 26, 256), (2 ** 34, 256),
])
def test_grid_covers_every_group_within_32_bits(tmp_path, n, threads):
    src = tmp_path / "g.cpp"
    src.write_text('#include "launch_grid.h"\n#include <cstdio>\n#include <cstdlib>\nint main(int, char **v) {'
                   "const rs::GroupGrid g = rs::group_grid(atoll(v[1]), atoi(v[2])); printf(\"%u %u\\n\", g.x, g.y); }\n")
    exe = tmp_path / "g"
    subprocess.check_call(["g++", "-I", CSRC, str(src), "-o", str(exe)])
    x, y = (int(v) for v in subprocess.check_output([str(exe), str(n), str(threads)], text=True).split())
    assert x * threads < 2 ** 32 and y < 65536
    assert n <= x * y < n + 8 * y
    if n * threads < 2 ** 32:
        assert (x, y) == (n, 1)
    else:
        assert x % 8 == 0
