"""The row ranges of the generic factor kernel, counted on the CPU (generic_plan_check.cpp)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_row_ranges_stay_short(tmp_path):
    exe = str(tmp_path / "generic_plan_check")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O2",
                    "-I", os.path.join(HERE, "..", "include"), os.path.join(HERE, "generic_plan_check.cpp"), "-o", exe], check=True, capture_output=True)
    done = subprocess.run([exe], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout == "0 faults\n", done.stdout
