"""The schedule of the blocked inversion, played on the CPU: no launch reads what another workgroup of it writes, every panel and tile
is up to date where it is read, and the result is the inverse."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "inverse_plan_check")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O2",
                    os.path.join(HERE, "inverse_plan_check.cpp"), "-o", exe], check=True, capture_output=True)
    return exe


# every matrix of up to 8,192 columns, and the largest that the entry points take (32,768 columns)
@pytest.mark.parametrize("blocks", [(2, 64), (127, 130), (253, 256)])
def test_no_launch_reads_what_it_writes(checker, blocks):
    done = subprocess.run([checker, *map(str, blocks)], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout.endswith(" 0 faults\n"), done.stdout
