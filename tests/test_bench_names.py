"""The kernel names the bench looks its measured counters up by are kernels of
the built library."""
import shutil
import subprocess

import pytest

import bench
from paper_1603_02655_amd import tc

TUNING = dict(hub_tile=1024, wave_tile=1024, group_size=256, group_tile=4096)


def test_instance_names_exist():
    if not shutil.which("nm"):
        pytest.skip("nm not available")
    out = subprocess.run(["nm", "-C", tc.LIB_PATH], capture_output=True, text=True, check=True).stdout
    kernels = {line.split("__device_stub__")[1].split("(")[0] for line in out.splitlines() if "__device_stub__" in line}
    for tri, names in ((True, ("k_tri_lane", "k_tri_wave", "k_tri_group", "k_tri_hub", "k_census_rows")),
                       (False, ("k_census_lane", "k_census_wave", "k_census_group", "k_census_hub"))):
        for name in names:
            assert bench.instance_name(name, tri, TUNING) in kernels
