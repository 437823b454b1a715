"""The committed records of the direct sum also belong to the committed headers that its kernels include (no GPU)."""
import hashlib
import json
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name", ["traffic.json", "k_direct_isa_mix.json"])
def test_headers_match(name):
    rec = json.load(open(os.path.join(ROOT, "profiles", name)))
    rec = rec.get("k_direct", rec)
    seen, todo = set(), [os.path.join(ROOT, rec["source"])]
    while todo:                                       # the source's own headers, wherever they are included from
        for h in re.findall(r'#include "([^"]+)"', open(todo.pop()).read()):
            path = os.path.join(ROOT, os.path.dirname(rec["source"]), h)
            if os.path.exists(path) and h not in seen:
                seen.add(h)
                todo.append(path)
    assert {os.path.basename(p) for p in rec["headers_sha256"]} == seen
    for path, digest in rec["headers_sha256"].items():
        assert hashlib.sha256(open(os.path.join(ROOT, path), "rb").read()).hexdigest() == digest, path


def test_bench_takes_the_records():
    import bench
    for name in ("traffic.json", "k_direct_isa_mix.json"):
        rec = json.load(open(os.path.join(ROOT, "profiles", name)))
        rec = rec.get("k_direct", rec)
        assert bench.record_current(rec)
        changed = dict(rec, headers_sha256={p: "0" for p in rec["headers_sha256"]})
        assert not bench.record_current(changed)
