"""Rules of the launch planner on the CPU under the address and undefined-behaviour sanitizers (see
plan_rules_harness.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.timeout(300)
def test_plan_rules_under_sanitizers(tmp_path):
    exe = tmp_path / "rules"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror",
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer",
                    "-I", os.path.join(ROOT, "paper_2602_23067_amd", "csrc"),
                    os.path.join(ROOT, "tests", "plan_rules_harness.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=250)
    assert out.returncode == 0, out.stderr[-4000:]
    assert "OK" in out.stdout
