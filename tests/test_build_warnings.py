"""The sorts' kernels build without warnings: the compiler warns where a launch
bound asks for more wavefronts than a kernel's LDS or registers allow."""
import os
import subprocess

from paper_2005_04680_amd import build


def test_launch_bounds_are_met(tmp_path):
    src = os.path.join(build.HERE, "csrc", "sort_tables.hip")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-c", src, "-o",
                        str(tmp_path / "sort_tables.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert "warning" not in r.stderr, r.stderr
