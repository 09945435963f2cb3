"""The host rules that cut a call into launch sequences (csrc/launch_rules.h), over their whole range in a plain C++
program."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_launch_rules_over_their_range(tmp_path):
    exe = str(tmp_path / "launch_rules")
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", exe, os.path.join(HERE, "c", "launch_rules.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, f"exit {r.returncode}: {r.stdout}{r.stderr}"
