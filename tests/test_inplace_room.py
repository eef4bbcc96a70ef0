"""In-place launches keep within the workspace's room for halo copies, for every
plan that the library can come to (host code only: runs without a GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_in_place_launch_fits_its_room(tmp_path):
    """Sizes 1..100001, every depth, storage type, default and chosen segment
    heights, all remainders from both layouts: the copies of each launch fit the
    room of lbm_workspace_bytes_inplace_blocked; twelve steps are among them."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "halo_room")
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17",
                    "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2208_14870_amd", "csrc"),
                    "-o", exe, os.path.join(ROOT, "tests", "halo_room.cpp")],
                   check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    words = r.stdout.split()
    assert int(words[words.index("plans") + 1]) > 100000
    assert int(words[words.index("deep") + 1]) > 1000
