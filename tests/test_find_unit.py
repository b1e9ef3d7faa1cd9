"""Which item a workgroup of the packed kernel takes without a work list: the kernel's own index arithmetic, compiled for the host and
walked for every workgroup of some 600 batches (CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_every_item_is_taken_once(tmp_path):
    exe, parts = tmp_path / "find_unit_check", 6
    # (the lanes' contexts jump between stacks, which a checked longjmp refuses)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Wno-unknown-pragmas", "-U_FORTIFY_SOURCE",
                           os.path.join(ROOT, "tests", "find_unit_check.cpp"), "-o", str(exe)])
    runs = [subprocess.Popen([str(exe), str(i), str(parts)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True) for i in range(parts)]
    for run in runs:
        out, _ = run.communicate(timeout=300)
        assert run.returncode == 0 and out.strip().endswith("ok"), out
