"""Chunk plans whose products run as two column tiles where that spares the fullest compute unit: which widths of which plans
(on stand-ins for the device).  The products are compared in test_gpu_halved_tiles.py."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2506_15174_amd", "csrc")


def test_two_tiles_where_their_own_order_spares_enough(tmp_path):
    exe = str(tmp_path / "halved_tiles")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-I", HERE,
                    "-I", os.path.join(rocm, "include"), os.path.join(HERE, "halved_tiles_on_stand_ins.cpp"),
                    os.path.join(CSRC, "spmm_api.cpp"), os.path.join(CSRC, "spmm_plan.cpp"), "-pthread", "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.endswith("ok\n"), res.stdout + res.stderr
