"""bench.py's measured traffic is that of the kernel that ran: a counter summary
of this source but of the other condensation kernel is not reported."""
import hashlib
import json
import os

import pytest

torch = pytest.importorskip("torch")

import bench


@pytest.mark.parametrize("ran", ["kb_prep_tile+kb_dm_finish", "kb_prep_band+kb_dm_finish"])
def test_traffic_of_the_kernel_that_ran(tmp_path, ran):
    with open(os.path.join(bench.ROOT, "paper_2510_12053_amd", "csrc", "cc_kernels.hip"), "rb") as f:
        source = hashlib.sha256(f.read()).hexdigest()[:16]
    rec = {"kernel": "kb_prep_tile+kb_dm_finish", "source_sha256_16": source}
    path = tmp_path / "traffic.md"
    path.write_text("traffic_json: " + json.dumps(rec) + "\n")
    assert bench.measured_traffic(str(path), ran) == (rec if ran == rec["kernel"] else None)
