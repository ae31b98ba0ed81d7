"""bench.py's lookup of the committed counter summaries (no GPU)."""
import json
import os
import re

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("kernel,prec", [("march_kernel", "fp32"), ("march_kernel", "fp64"), ("step3_kernel", "fp32"),
                                         ("step3_kernel", "fp64"), ("step2_kernel", "fp16s")])
def test_the_default_kernels_have_a_counter_summary(kernel, prec, monkeypatch):
    """The summary of each 2048^2 kernel lies where bench.py looks, and its traffic is reported for the
    launch and the kernel code that it was taken with, and for no other."""
    text = open(os.path.join(ROOT, "profiles", f"{kernel}_{prec}_cavity2048.md")).read()
    d = json.loads(re.search(r"```json\n(.*?)\n```", text, re.S).group(1))
    monkeypatch.setattr(bench, "kernel_code_hash", lambda: d["kernel_code_sha256_16"])
    assert bench.profiled_traffic(prec, 2048, d["launch"] + [kernel]) == d["traffic_bytes_per_launch"] > 0
    assert bench.profiled_traffic(prec, 2048, [64, 1] + d["launch"][2:] + [kernel]) is None
    monkeypatch.setattr(bench, "kernel_code_hash", lambda: "other")
    assert bench.profiled_traffic(prec, 2048, d["launch"] + [kernel]) is None
