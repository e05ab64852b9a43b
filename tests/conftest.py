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
def oracle():
    import oracle as _oracle
    _oracle.build()
    return _oracle


@pytest.fixture(autouse=True)
def _no_garbage_from_earlier_tests(request):
    """A test that counts allocated device memory starts without tensors that earlier tests left in reference cycles
    (a caught exception's traceback): the collector may free those at any point of it."""
    if request.module.__name__ == "test_zz_no_alloc":
        gc.collect()
    yield
