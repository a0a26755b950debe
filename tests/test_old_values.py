"""Where the factor tiles ask for the old values of a running average, counted on the CPU (old_values_check.cpp)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_old_values_lie_inside_the_matrix(tmp_path):
    exe = str(tmp_path / "old_values_check")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O2",
                    "-I", os.path.join(HERE, "..", "include"), os.path.join(HERE, "old_values_check.cpp"), "-o", exe], check=True, capture_output=True)
    done = subprocess.run([exe], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout == "0 faults\n", done.stdout
