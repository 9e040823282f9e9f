"""Every kernel launch that the library's host code makes is linked to it: none
is weak, so a build that lost one fails instead of going another way."""

import os
import shutil
import subprocess

import pytest

OBJ = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_11709_amd", "_build", "api.o")


@pytest.mark.skipif(shutil.which("nm") is None or not os.path.exists(OBJ), reason="nm or the built object not there")
def test_no_weak_launches():
    lines = subprocess.run(["nm", "-C", OBJ], capture_output=True, text=True, check=True).stdout.splitlines()
    launches = [l for l in lines if "xrd::launch_" in l]
    assert len(launches) > 10
    assert not [l for l in launches if l.split()[0].lower() in ("w", "v")]
