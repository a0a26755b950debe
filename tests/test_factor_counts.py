"""What the factor builds work out in whole numbers, counted on the CPU: where old values of a running average are asked for, the generic
kernel's row ranges, and the scratch of builds in calls of every kind."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.parametrize("check", ["old_values_check", "generic_plan_check", "call_cut_check"])
def test_no_faults(check, tmp_path):
    exe = str(tmp_path / check)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O2",
                    "-I", os.path.join(HERE, "..", "include"), os.path.join(HERE, check + ".cpp"), "-o", exe], check=True, capture_output=True)
    done = subprocess.run([exe], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout == "0 faults\n", done.stdout
