"""bench.py's roofline block on the CPU: the HBM-traffic constant of whole
one-kernel steps is the figure the committed rocprofv3 summary states, and its
label names that summary."""
import os
import re

from test_bench_contract import ROOT, _bench_module


def test_step_traffic_constant_matches_the_profile():
    b = _bench_module()
    name = "step_kernel_c3_first_steps_hbm_traffic.md"
    text = open(os.path.join(ROOT, "profiles", name)).read()
    m = re.search(r"\*\*([0-9.]+) bytes per particle-step\*\*", text)
    assert m and float(m.group(1)) == b.STEP_TRAFFIC_BYTES_PER_PARTICLE
    assert name in b.STEP_TRAFFIC_SOURCE
