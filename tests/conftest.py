import os
import shutil
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def golden_dir():
    return os.path.join(ROOT, "tests", "golden")


@pytest.fixture(scope="session")
def recording_library(tmp_path_factory):
    """The library's host code on a runtime that records launches (tests/host_library.py)."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not installed")
    from tests import host_library
    return host_library.build(str(tmp_path_factory.mktemp("recording")))
