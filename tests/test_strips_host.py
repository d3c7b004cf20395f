"""The builder of the strips path, on the host (tests/strips_on_host.cpp)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2506_15174_amd", "csrc")


def test_strips_hold_every_entry_once(tmp_path):
    exe = str(tmp_path / "strips_on_host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, os.path.join(HERE, "strips_on_host.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.endswith("ok\n"), res.stdout + res.stderr
