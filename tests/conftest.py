import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import host_rules  # noqa: E402
import oracle      # noqa: E402


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")
    # Whatever has to be compiled for the tests is, before one of them starts the GPU: from then on no process is to be started (a run has
    # ended with a segmentation fault where g++ was, by the first test that asked for a host rule).
    host_rules.lib()
    oracle.lib()


def pytest_collection_modifyitems(config, items):
    # Printing the test id before each GPU test names the case if the box dies under it.
    pass


@pytest.fixture(autouse=True)
def _announce(request):
    if request.node.get_closest_marker("gpu"):
        print(f"\n[gpu-test] {request.node.nodeid}", flush=True)
    yield
