"""The attention schedule (csrc/attn_schedule.h, host code only): tests/host_san/schedule.cpp, built with sanitizers."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_key_tile_is_covered_once(tmp_path):
    exe = str(tmp_path / "schedule")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-static-libasan", os.path.join(ROOT, "tests", "host_san", "schedule.cpp"), "-o", exe])
    run = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-4000:]
    assert "attention schedule: ok" in run.stdout
