"""The memory traffic that bench.py reports is read from the committed counter summaries: each must name the kernel that the
workload runs."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402
from paper_2104_08378_amd import synth  # noqa: E402


@pytest.mark.parametrize("name", ["ffn_bf16", "square_i8", "skinny_bf16", "conv3x3_f16"])
def test_traffic_of_the_product_covers_its_operands(name):
    w = synth.WORKLOADS[name]
    es = 1 if w["dtype"] == "i8" else 2
    out = {"i32": 4, "f32": 4, "bf16": 2, "f16": 2}[w["out"]]
    b = 64 * 14 * 14 * 256 * 2 if name == "conv3x3_f16" else w["N"] * w["K"] * es          # the NHWC input, or B
    need = w["M"] * w["K"] // 2 * es + w["M"] * w["K"] // 8 + b + w["M"] * w["N"] * out
    assert need <= bench.measured_traffic(name) <= 3 * need
