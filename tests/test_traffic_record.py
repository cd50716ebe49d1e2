"""The committed traffic record names, for every kernel, the source file that
holds it (its hash there decides whether bench.py may quote the bytes)."""

import json
import os
import re

import bench


def test_sources_hold_the_kernels():
    with open(bench.TRAFFIC_FILE) as f:
        record = {k: v for k, v in json.load(f).items() if isinstance(v, dict)}
    assert "softmax_bf16_kernel<128,128,8,kFem>" in record
    for name, ent in record.items():
        src = os.path.join(bench.ROOT, "paper_2602_07160_amd", "csrc", ent["source"])
        with open(src) as f:
            code = f.read()
        assert re.search(r"__global__[^;{]*\b" + re.match(r"\w+", name)[0] + r"\(", code), name
