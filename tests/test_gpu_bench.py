"""bench.py's measurement of one workload on the device: the record names the
kernel that ran, and holds figures for it, however short the warm-up."""
import math
import os
import sys

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("warmup", [1, 3])
def test_record_of_one_short_session(warmup):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    import bench
    from synth import configs as C
    rec, _, _ = bench.measure(C.with_overrides(C.get("small"), steps=8), warmup, 3, torch.device("cuda:0"))
    assert rec["roofline"]["kernel"] == "k_rows" and rec["roofline"]["launches"] == 3
    assert math.isfinite(rec["roofline"]["achieved"]) and rec["value"] > 0
    assert rec["observe_path"]["first"] == rec["observe_path"]["steady"] == "session"
