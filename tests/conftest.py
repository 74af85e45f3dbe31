import gc
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu on the GPU box)")


@pytest.fixture(scope="session")
def hero():
    """The HIP library binding; GPU tests fail loudly if it cannot be loaded."""
    import paper_2310_17723_amd as pkg
    return pkg.load()


@pytest.fixture(autouse=True, scope="module")
def _garbage_of_the_module_before():
    """A pytest.raises block ties its frame into a cycle, the test's device tensors with it: collected here, not in the middle of a
    test that counts device memory."""
    gc.collect()
