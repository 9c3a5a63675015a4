"""rg_plan and rg_plan_f32w say what rg_linear, rg_linear_bias and rg_linear_f32w launch (kernel, tile, waves,
workgroups), for every kernel and override, and a launch the runtime refuses is an error, never another kernel
(tests/asan/dispatch_harness.cpp: the library's rg_api.cpp with stubbed launchers; no device)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plan_reports_what_is_launched(tmp_path):
    from paper_2609_25624_amd import build as b
    if not os.path.exists(b.HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "dispatch_harness")
    cmd = [b.HIPCC, "-x", "hip", "-std=c++17", "-O1", *b.DEVICE,
           os.path.join(ROOT, "paper_2609_25624_amd", "csrc", "rg_api.cpp"),
           os.path.join(ROOT, "tests", "asan", "dispatch_harness.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok:"), (r.returncode, r.stdout[-2000:], r.stderr[-2000:])
