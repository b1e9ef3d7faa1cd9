import ctypes
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_collection_modifyitems(config, items):
    import torch

    if torch.cuda.is_available():
        return
    skip = pytest.mark.skip(reason="no GPU in this process")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


@pytest.fixture(scope="session")
def batch_rules(tmp_path_factory):
    """The library's own rules for which form a batch takes (csrc/batch_rules.hpp), compiled for the host."""
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    lib = tmp_path_factory.mktemp("rules") / "batch_rules.so"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-shared", "-fPIC", os.path.join(ROOT, "tests", "batch_rules_check.cpp"), "-o", str(lib)])
    return ctypes.CDLL(str(lib))
