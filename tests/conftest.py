import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: test needs a real MI355X (runs the HIP library)")


@pytest.fixture(autouse=True, scope="module")
def no_garbage_left():
    """Tensors in reference cycles (a caught error's frames) go with their module, not under a later test that counts
    memory."""
    yield
    gc.collect()
