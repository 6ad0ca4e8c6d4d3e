"""The planner that cuts the last round of an attention launch of equal work items, checked on the host (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tail_plan_covers_every_block_once(tmp_path):
    exe = tmp_path / "attn_tail_check"
    src = os.path.join(ROOT, "tests", "host", "attn_tail_check.cpp")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined", src, "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
